// K loops for tall tiles of the expert GEMMs (which tiles: takes_tall_loop); included by moe_gemm_kernel.hpp, which
// describes what all tiles share.  First the fp8 loop; what the bf16 loop does otherwise stands before it.
//
// In gemm_tile every wavefront reads all token rows of a K step from LDS and its own weight rows, and a step is a
// chain: barrier, first fragments from LDS, MFMAs that each wait for the scales of the one before.  For a tile of
// 16 row blocks that is 288 KiB of fragment reads per step and the matrix cores busy a third of the time (with all
// copies switched off the launch still took 83 % of its time).  Here the eight wavefronts form a grid, two along the
// token rows and four along the weight rows (192 KiB of fragment reads), and the step is a pipeline:
//  * the product of MFMA i is folded into the sums behind MFMA i + 2;
//  * the one barrier of a step sits before its last six MFMAs.  It opens the next stage, whose fragments are read
//    into registers as the last MFMAs of this one set them free, and gives up this one, whose place the copies of the
//    step after next take.  They are issued one by one between MFMAs: in one go they would hold the wavefront up;
//  * token scales come four K steps at a time, 16 bytes per row, a quarter of the rows with each step: a quarter of
//    the requests of one 4-byte copy per row and step (those were 30 % of all L2 requests);
//  * LDS row r holds 16-byte chunk c at place c ^ (r & 7) ^ (r >> 3 & 1): with c ^ (r & 7) alone the sixteen lanes that a
//    16-byte read serves at a time meet in pairs (bank conflicts of 6.6e7 LDS cycles in 1.5e8 of the launch below; with
//    the loop as a whole 1.2e7 in 0.7e8).
// The sums see the same terms in the same order as in gemm_tile (rotated starts apart: whole blocks of four steps).
// Measured on the 32-expert share of the DeepSeek-shaped layer: 16384 tokens, gate/up 612 -> 498 us, down 346 -> 317;
// 4096 tokens, 228 -> 222 and 133 -> 123.
// Fetching the lines of three steps ahead into L2 as well was slower (498 -> 553): the requests cost more than the
// latency they hide.  Other tiles and half-width items go through gemm_tile.
#pragma once
#include <type_traits>

namespace moe {
namespace {

// LDS of a tall fp8 tile: two stages of token rows, two of weights, three blocks of four steps' token scales
template <class SH>
struct Tall8 {
    static constexpr int A_STAGE = 256 * 128, W_STAGE = 256 * 128, SC_BLOCK = 256 * 16;
    static constexpr int W_RING = 2 * A_STAGE, SC_RING = W_RING + 2 * W_STAGE;
    static constexpr int LDS_BYTES = SC_RING + 3 * SC_BLOCK;
    static_assert(LDS_BYTES <= SH::LDS_BYTES, "the launch reserves it");
};

// What a wavefront knows about its tile.
struct TallArgs {
    const GemmArgs &g;
    const moe_tile &tile;
    unsigned char *smem;
    int tid, wave, ct, nk, koff;
};

// One wavefront's part of a tall tile: NBT (4..8) blocks of 16 token rows, the first of them block TB0 of the
// tile's NB, times 64 weight rows (gate/up: 32 gate rows and the matching up rows).
template <class SH, int NB, int NBT, int TB0, bool SHARE>
__device__ __forceinline__ void tall8_wave(const TallArgs &t)
{
    using TL = Tall8<SH>;
    constexpr bool SWIGLU = SH::SWIGLU;
    constexpr int NW = SH::NW, WB = 4;
    constexpr int A_PASS = (2 * NB + NW - 1) / NW;            // 8-row token copies per wavefront and step
    constexpr int W_PASS = 4;                                 // 8-row weight copies per wavefront and step
    constexpr int NCOPY = 1 + A_PASS + W_PASS;                // scales, tokens, weights
    constexpr int NPRE = 6;                                   // of these, issued in the step before
    static_assert(NBT >= 4 && 2 * (NBT - 2) >= NCOPY - NPRE, "the copies of a step are issued before its meeting");

    const GemmArgs &g = t.g;
    const moe_tile &tile = t.tile;
    unsigned char *const smem = t.smem;
    const int lane = t.tid & 63, wave = t.wave, ct = t.ct, nk = t.nk, wn = wave & 3;
    const int l16 = lane & 15, lq = lane >> 4;
    const int crow = lane >> 3;
    // LDS row r holds logical 16-byte chunk c at place c ^ (r & 7) ^ (r >> 3 & 1): the sixteen lanes that a
    // 16-byte fragment read serves at a time then cover all banks
    const int cbyte = ((lane & 7) ^ crow) << 4;
    const int rows = tile.rows, n_out = g.n_out, w_rows = SWIGLU ? 2 * n_out : n_out;
    const size_t row_bytes = (size_t)g.K;

    // this wavefront's weight scales for every K step, lane l holds step l (and l + 64)
    float wsc[SWIGLU ? 2 : 1][2];
    {
        const int cc = min(ct * SH::COLS + wn * (SH::COLS / 4), n_out - 1);
#pragma unroll
        for (int j = 0; j < (SWIGLU ? 2 : 1); ++j) {
            const float *ws = g.w_scale + ((size_t)tile.expert * (w_rows / kQBlock) + (j * n_out + cc) / kQBlock) * nk;
            wsc[j][0] = ws[min(lane, nk - 1)];
            wsc[j][1] = ws[min(lane + 64, nk - 1)];
        }
    }

    // this wavefront moves weight rows 32*wave .. 32*wave+31 of the stage (a quarter of the gate/up slab
    // holds its 32 gate rows, then the matching up rows) ...
    const int wcol0 = ct * SH::COLS + (SWIGLU ? (wave >> 1) * 32 : wave * 32);
    const int wc0 = __builtin_amdgcn_readfirstlane(min(wcol0, n_out - 1));
    const unsigned char *const w_base = g.W + ((size_t)tile.expert * w_rows + (SWIGLU && (wave & 1) ? n_out : 0) + wc0) * row_bytes;
    uint32_t w_off[W_PASS];
#pragma unroll
    for (int q = 0; q < W_PASS; ++q)                          // columns past the end repeat the last one; never stored
        w_off[q] = (uint32_t)(min(wcol0 + q * 8 + crow, n_out - 1) - wc0) * (uint32_t)row_bytes + (cbyte ^ (q & 1) * 16);
    // ... token rows 8*(wave + 8 i) .. +7, and of the first four wavefronts the scales of rows 64*wave .. +63
    auto src_row = [&](int r) __attribute__((always_inline)) -> size_t {
        r = min(r, rows - 1);                                 // padded rows repeat the last row; never stored
        if constexpr (SWIGLU) return (size_t)(g.sorted_pair[tile.row0 + r] / g.top_k);
        else return (size_t)(tile.row0 + r);
    };
    const unsigned char *a_ptr[A_PASS];
#pragma unroll
    for (int i = 0; i < A_PASS; ++i)
        a_ptr[i] = g.A + src_row(8 * (wave + NW * i) + crow) * row_bytes + (cbyte ^ (wave & 1) * 16);
    const float *const sc_ptr = g.a_scale + src_row((wave & 3) * 64 + lane) * nk;
    // the scales have arrived with the addresses above: said here, so that nothing waits for them inside the loop
#pragma unroll
    for (int j = 0; j < (SWIGLU ? 2 : 1); ++j) asm volatile("" : "+v"(wsc[j][0]), "+v"(wsc[j][1]));
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr_of(smem));
    const uint32_t a_lds = lds0 + wave * 1024, w_lds = lds0 + TL::W_RING + wave * (W_PASS * 1024);
    const uint32_t sc_lds = lds0 + TL::SC_RING + (wave & 3) * 1024;

    f32x4 acc[NBT][WB];
#pragma unroll
    for (int m = 0; m < NBT; ++m)
#pragma unroll
        for (int b = 0; b < WB; ++b) acc[m][b] = f32x4{0.f, 0.f, 0.f, 0.f};

    // state of the copies: stage that they fill next (K step after rotation, LDS places)
    int kc = t.koff;
    uint32_t stage_off = 0;                                   // 0 or one stage
    int sc_off = 0;                                           // ring place of the scale block after kc's
    auto copy = [&](int c) __attribute__((always_inline)) {   // copy c of NCOPY of the stage
        const int k0 = kc * GM_STEP_BYTES;
        if (c == 0) {
            // a quarter of the next four steps' scales rides with each stage of the block before
            const int blk = (kc >> 2) + 1;
            copy16_to_lds_if(wave ^ (kc & 3), sc_ptr + (blk * 4 == nk ? 0 : blk * 4), sc_lds + sc_off);
        } else if (c <= A_PASS) {
            copy16_to_lds<false>(a_ptr[c - 1] + k0, a_lds + stage_off + (c - 1) * (NW * 1024));
        } else {
            const int q = c - 1 - A_PASS;
            copy16_to_lds_at<!SHARE>(w_base + k0, w_off[q], w_lds + stage_off + q * 1024);
            if (q == W_PASS - 1) {                            // the stage is complete: on to the next
                if ((kc & 3) == 3) sc_off = sc_off == 2 * TL::SC_BLOCK ? 0 : sc_off + TL::SC_BLOCK;
                kc = kc + 1 == nk ? 0 : kc + 1;
                stage_off ^= TL::A_STAGE;
            }
        }
    };

    // a fragment is two neighbouring chunks: the second one's place is the first's with bit 4 flipped
    const int chunk = ((2 * lq) ^ (l16 & 7) ^ (l16 >> 3)) << 4;
    const int to = TB0 * 2048 + l16 * 128 + chunk, to2 = to ^ 16;
    const int wo = TL::W_RING + wn * 8192 + l16 * 128 + chunk, wo2 = wo ^ 16;
    int cur = 0;                                              // stage being computed: 0 or one stage
    // Token block m of a wavefront uses register set slot(m): two sets in turn, three where the last block but
    // one would otherwise not meet set 0 (the next step starts with set 0, free first).
    constexpr int TS = (NBT & 1) ? 3 : 2;
    auto slot = [](int m) constexpr { return (NBT & 1) && m >= NBT - 3 ? (m - (NBT - 3) + 2) % 3 : m & 1; };
    i32x8 wq[WB], tf[TS];
    float ts[TS];
#define MOE_FRAG8(off_, off2_, imm_) ({ const u32x4 lo_ = *reinterpret_cast<const u32x4 *>(smem + (off_) + (imm_)); \
                           const u32x4 hi_ = *reinterpret_cast<const u32x4 *>(smem + (off2_) + (imm_)); \
                           i32x8{(int)lo_.x, (int)lo_.y, (int)lo_.z, (int)lo_.w, (int)hi_.x, (int)hi_.y, (int)hi_.z, (int)hi_.w}; })
#define MOE_WGT8(b_, st_) wq[b_] = MOE_FRAG8(wo + (st_), wo2 + (st_), (b_) * 2048);
#define MOE_TOK8(m_, st_, so_) { tf[slot(m_)] = MOE_FRAG8(to + (st_), to2 + (st_), (m_) * 2048); ts[slot(m_)] = *reinterpret_cast<const float *>(smem + (so_) + (m_) * 256); }

    // stage 0 with the first scale block, then the start of stage 1
    if (wave < 4) copy16_to_lds<false>(sc_ptr + (kc & ~3), sc_lds + 2 * TL::SC_BLOCK);
#pragma unroll
    for (int c = 0; c < NCOPY; ++c) copy(c);
    if (nk > 1) {
#pragma unroll
        for (int c = 0; c < NPRE; ++c) copy(c);
    }
    // (a wavefront that copied no scales has issued one less than NPRE)
    if (nk > 1) MOE_WAIT_VMCNT(NPRE - 1);
    else MOE_WAIT_VMCNT(0);
    asm volatile("s_barrier" ::: "memory");
    int kr = t.koff;                                          // K step (after rotation) being computed
    int so = TL::SC_RING + 2 * TL::SC_BLOCK + TB0 * 256 + l16 * 16 + (kr & 3) * 4;
#pragma unroll
    for (int b = 0; b < WB; ++b) MOE_WGT8(b, 0)
    MOE_TOK8(0, 0, so)
    MOE_TOK8(1, 0, so)
    __builtin_amdgcn_sched_barrier(0);

    // LEFT: steps after this one: 0, 1, or 2 (two and more)
    auto step = [&](auto left_) __attribute__((always_inline)) {
        constexpr int LEFT = decltype(left_)::value;
        const int next = cur ^ TL::A_STAGE;
        const int kn = kr + 1 == nk ? 0 : kr + 1;
        // the next step's place in the scale ring
        int so_next = so + 4;
        if ((kr & 3) == 3) {
            so_next = so - 12 + TL::SC_BLOCK;
            if (so_next >= TL::SC_RING + 3 * TL::SC_BLOCK) so_next -= 3 * TL::SC_BLOCK;
        }
        float sw[SWIGLU ? 2 : 1];
#pragma unroll
        for (int j = 0; j < (SWIGLU ? 2 : 1); ++j)
            sw[j] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, kr < 64 ? wsc[j][0] : wsc[j][1]), kr & 63));

        // The products of MFMA i are folded into the sums while MFMA i + 2 runs.
        f32x4 pp[3];
        float fs[TS][2];                                      // [token block's register set][gate / up]
        constexpr int NM = NBT * WB;
        // MFMA i of the step: its token block and weight block.  All weight blocks of a token block in
        // turn; the last two token blocks, X and Y, go side by side, so that the weights are done with one by one.
        constexpr int X = NBT - 2, Y = NBT - 1;
        constexpr int TAIL_M[8] = {X, X, Y, X, Y, X, Y, Y}, TAIL_B[8] = {0, 1, 0, 2, 1, 3, 2, 3};
        auto m_of = [&](int i) constexpr { return i < NM - 8 ? i / WB : TAIL_M[i - (NM - 8)]; };
        auto b_of = [&](int i) constexpr { return i < NM - 8 ? i % WB : TAIL_B[i - (NM - 8)]; };
#pragma unroll
        for (int i = 0; i < NM + 2; ++i) {
            if (i < NM) {
                const int m = m_of(i), b = b_of(i);
                const f32x4 zero = f32x4{0.f, 0.f, 0.f, 0.f};
                // e4m3 x e4m3, hardware block scales set to 1.0 (E8M0 0x7f): the fp32 scales are applied below
                pp[i % 3] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(wq[b], tf[slot(m)], zero, 0, 0, 0, 0x7f7f7f7f, 0, 0x7f7f7f7f);
                if (b == 0) {
#pragma unroll
                    for (int j = 0; j < (SWIGLU ? 2 : 1); ++j) fs[slot(m)][j] = ts[slot(m)] * sw[j];
                }
            }
            if (i >= 2) {
                const int pm = m_of(i - 2), pb = b_of(i - 2);
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    acc[pm][pb][v] = fmaf(pp[(i - 2) % 3][v], fs[slot(pm)][SWIGLU ? pb >> 1 : 0], acc[pm][pb][v]);
            }
            if (i < NM - 8) {
                if (i % WB == WB - 1) {                       // the token block is done with: fetch the one after next
                    const int m = i / WB;
                    if (m + 2 < NBT) MOE_TOK8(m + 2, cur, so)
                }
                if (LEFT >= 1 && (i & 1) == 0 && NPRE + i / 2 < NCOPY) copy(NPRE + i / 2);
            } else if (LEFT >= 1) {
                const int j = i - (NM - 8);
                if (j == 1) {
                    // every fragment of this stage has been requested: once they are here, and the next stage
                    // has landed, all wavefronts meet; then this stage may be overwritten
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    MOE_WAIT_VMCNT(0);
                    asm volatile("s_barrier" ::: "memory");
                }
                if (j == 2) MOE_WGT8(0, next)
                if (j == 4) MOE_WGT8(1, next)
                if (j == 5) MOE_TOK8(0, next, so_next)
                if (j == 6) MOE_WGT8(2, next)
                if (j == 7) { MOE_WGT8(3, next) MOE_TOK8(1, next, so_next) }
                if (LEFT >= 2 && j >= 2 && j - 2 < NPRE) copy(j - 2);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        cur = next;
        so = so_next;
        kr = kn;
    };
    for (int s = 0; s + 2 < nk; ++s) step(std::integral_constant<int, 2>{});
    if (nk > 1) step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 0>{});
    MOE_WAIT_VMCNT(0);                                        // (nothing is in flight; cheap insurance for the LDS reuse below)
#undef MOE_TOK8
#undef MOE_FRAG8

    // ---- epilogue, as in gemm_tile: the output tile is staged in LDS and leaves as whole rows
    constexpr int OUT_ES = SWIGLU ? 1 : 2;
    constexpr int ROW_B = SH::COLS * OUT_ES, CPR = ROW_B / 16;
    constexpr int RED_BYTES = SWIGLU ? 4 * NB * 16 * 4 : 0;
    static_assert(RED_BYTES + NB * 16 * ROW_B <= TL::LDS_BYTES, "output tile must fit the LDS of the rings");
    unsigned char *const stage = smem + RED_BYTES;
    auto stage_at = [&](int r, int byte) __attribute__((always_inline)) {
        return stage + r * ROW_B + ((((byte >> 4) ^ ((r & (CPR / 2 - 1)) << 1))) << 4) + (byte & 15);
    };
    const int wcol = wn * (SH::COLS / 4);
    __syncthreads();
    if constexpr (SWIGLU) {
        float *const red = reinterpret_cast<float *>(smem);   // [4][NB*16]
        float a[NBT][2][4];
#pragma unroll
        for (int m = 0; m < NBT; ++m) {
            float mx = 0.f;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float gt = acc[m][j][v], up = acc[m][2 + j][v];
                    a[m][j][v] = gt / (1.f + __expf(-gt)) * up;
                    mx = fmaxf(mx, fabsf(a[m][j][v]));
                }
            mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
            mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
            if (lq == 0) red[wn * (NB * 16) + (TB0 + m) * 16 + l16] = mx;
        }
        __syncthreads();
#pragma unroll
        for (int m = 0; m < NBT; ++m) {
            const int r = (TB0 + m) * 16 + l16;
            float amax = 0.f;
#pragma unroll
            for (int wv = 0; wv < 4; ++wv) amax = fmaxf(amax, red[wv * (NB * 16) + r]);
            const float scale = amax > 0.f ? amax / GM_FP8_MAX : 1.f;
            const float inv = 1.f / scale;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                float q[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) q[v] = fminf(fmaxf(a[m][j][v] * inv, -GM_FP8_MAX), GM_FP8_MAX);
                int packed = 0;
                packed = __builtin_amdgcn_cvt_pk_fp8_f32(q[0], q[1], packed, false);
                packed = __builtin_amdgcn_cvt_pk_fp8_f32(q[2], q[3], packed, true);
                *reinterpret_cast<int *>(stage_at(r, wcol + j * 16 + lq * 4)) = packed;
            }
            if (r < rows && wn == 0 && lq == 0) g.out_scale[(size_t)(tile.row0 + r) * (n_out / kQBlock) + ct] = scale;
        }
    } else {
#pragma unroll
        for (int m = 0; m < NBT; ++m)
#pragma unroll
            for (int b = 0; b < WB; ++b) {
                uint2 o;
                o.x = pack_bf16x2(acc[m][b][0], acc[m][b][1]);
                o.y = pack_bf16x2(acc[m][b][2], acc[m][b][3]);
                *reinterpret_cast<uint2 *>(stage_at((TB0 + m) * 16 + l16, (wcol + b * 16 + lq * 4) * 2)) = o;
            }
    }
    __syncthreads();
    const size_t out_pitch = (size_t)n_out * OUT_ES;
    for (int c = t.tid; c < rows * CPR; c += SH::THREADS) {
        const int r = c / CPR, ch = c % CPR;
        const int col = ct * SH::COLS + ch * (16 / OUT_ES);
        if (col < n_out) {
            const u32x4 v = *reinterpret_cast<const u32x4 *>(stage_at(r, ch * 16));
            u32x4 *dst = reinterpret_cast<u32x4 *>(g.out + (size_t)(tile.row0 + r) * out_pitch + (size_t)col * OUT_ES);
            if (g.nt_out) __builtin_nontemporal_store(v, dst);
            else *dst = v;
        }
    }
}

// A tall tile of NB row blocks by a workgroup of eight wavefronts.  The first four take the first (NB+1)/2 row
// blocks, the others the rest: each of a compute unit's four matrix pipes holds one wavefront of either half.
template <class SH, int NB, bool SHARE>
__device__ __forceinline__ void gemm_tile_tall8(const GemmArgs &g, const Item &item, unsigned char *smem)
{
    int tid_opaque = threadIdx.x;                             // (see gemm_tile)
    asm volatile("" : "+v"(tid_opaque));
    const int nk = g.K / GM_STEP_BYTES;
    const int koff = (int)((long)(item.work % g.k_groups) * nk / g.k_groups) & ~3;   // whole scale blocks
    const int wave = __builtin_amdgcn_readfirstlane(tid_opaque >> 6);
    const TallArgs t{g, item.tile, smem, tid_opaque, wave, item.ct, nk, koff};
    constexpr int N0 = (NB + 1) / 2, N1 = NB / 2;
    if (wave < 4) tall8_wave<SH, NB, N0, 0, SHARE>(t);
    else tall8_wave<SH, NB, N1, N0, SHARE>(t);
}

// ---- bf16 ------------------------------------------------------------------------------------------------------
//
// Tall tiles of experts with three and more of them (long prompts on few experts: the matrix cores' regime).  The same
// grid of wavefronts and the same kind of step on v_mfma_f32_32x32x16_bf16: one wavefront alone issues 60 % of the
// 16x16x32 rate and all of this one, so a matrix pipe keeps busy while its other wavefront waits.  Fragments are
// requested PF groups of two MFMAs ahead; the barrier of a step sits before its last groups.  Weights have three
// stages of LDS (their lines come from HBM), token rows two.
// 4096 Mixtral tokens: gate/up 1708 -> 1658 us, down 866 -> 833 (a library GEMM of the same shape: 1615 for the
// gate/up part).  The clock is down to 1.62 to 1.67 GHz there: what is left is power more than cycles.
// Experts of one or two tiles stay with gemm_tile, in which a wavefront refills its own weights without a barrier: where
// the weight stream is the time it is the faster one (4096 DeepSeek tokens, gate/up 2736 us against 2793 with this loop
// for all tall tiles).  Few experts of two tiles would gain here (eight of 4096 x 14336 with 300 rows each, 622 -> 567).
typedef __attribute__((ext_vector_type(16))) float f32x16;

// LDS of a tall bf16 tile: two stages of token rows, three of weights.
template <class SH>
struct Tall16 {
    static constexpr int A_STAGE = 256 * 128, W_STAGE = 256 * 128;
    static constexpr int W_RING = 2 * A_STAGE;
    static constexpr int LDS_BYTES = W_RING + 3 * W_STAGE;
    static_assert(LDS_BYTES <= SH::LDS_BYTES, "the launch reserves it");
};

// What a wavefront of gemm_tile_tall16 knows about its tile.
struct Tall16Args {
    const GemmArgs &g;
    const moe_tile &tile;
    unsigned char *smem;
    int tid, lane, wave, ct, kh, nk, koff;
    size_t row_bytes, kbase;
};

// One wavefront's part: NBT blocks of 32 token rows (the first is block TB0 of the tile's TB) times 64 weight rows.
template <class SH, int TB, int NBT, int TB0>
__device__ __forceinline__ void tall16_wave(const Tall16Args &t)
{
    using TL = Tall16<SH>;
    constexpr bool SWIGLU = SH::SWIGLU;
    constexpr int NW = SH::NW, WB = 2;                        // 32-row weight blocks per wavefront
    constexpr int A_PASS = (4 * TB + NW - 1) / NW;            // 8-row token copies per wavefront and step
    constexpr int W_PASS = 4;                                 // 8-row weight copies per wavefront and step
    constexpr int NKK = 4;                                    // 16-wide MFMA steps of a K step
    constexpr int NQ = NKK * NBT;                             // token fragments (groups of WB MFMAs) of a step
    constexpr int PF = NBT > 1 ? 4 : 2;                       // fragments requested ahead
    static_assert(NQ % PF == 0, "a fragment keeps its registers from step to step");
    constexpr int QB = NQ - PF + 1;                           // group after which the next stage is opened
    static_assert(QB >= (NKK - 2) * NBT, "the last weight fragments are requested before the stage is given up");
    constexpr int CPG = (A_PASS + W_PASS + QB) / (QB + 1);    // copies issued per group: all of them before that point
    constexpr int NPRE = (NQ - QB) * CPG < A_PASS ? (NQ - QB) * CPG : A_PASS;   // token copies issued right after it

    const GemmArgs &g = t.g;
    const moe_tile &tile = t.tile;
    unsigned char *const smem = t.smem;
    const int lane = t.lane, wave = t.wave, ct = t.ct, nk = t.nk;
    const int wn = wave & 3;
    const int l32 = lane & 31, lh = lane >> 5;
    const int crow = lane >> 3;
    // LDS row r holds logical 16-byte chunk c at place c ^ (r & 7) ^ (r >> 3 & 1): the sixteen rows that a
    // 16-byte fragment read serves at a time then cover all banks
    const int cbyte = ((lane & 7) ^ crow) << 4;
    const int rows = tile.rows;
    const int n_out = g.n_out;
    const int w_rows = SWIGLU ? 2 * n_out : n_out;

    // weight copies: this wavefront moves LDS rows 32*wave .. 32*wave+31 of the stage.  A quarter of the
    // gate/up slab holds its 32 gate rows, then the matching up rows.
    const int wcol0 = ct * SH::COLS + (SWIGLU ? (wave >> 1) * 32 : wave * 32);     // first output column of these rows
    const int wc0 = __builtin_amdgcn_readfirstlane(min(wcol0, n_out - 1));
    const unsigned char *w_base = g.W + ((size_t)tile.expert * w_rows + (SWIGLU && (wave & 1) ? n_out : 0) + wc0) * t.row_bytes + t.kbase;
    uint32_t w_off[W_PASS];
#pragma unroll
    for (int q = 0; q < W_PASS; ++q)                          // columns past the end repeat the last one; never stored
        w_off[q] = (uint32_t)(min(wcol0 + q * 8 + crow, n_out - 1) - wc0) * (uint32_t)t.row_bytes + (cbyte ^ (q & 1) * 16);
    const unsigned char *a_ptr[A_PASS];
#pragma unroll
    for (int i = 0; i < A_PASS; ++i) {
        const int r = min(8 * (wave + NW * i) + crow, rows - 1);   // padded rows repeat the last row; never stored
        size_t src;
        if constexpr (SWIGLU) src = (size_t)(g.sorted_pair[tile.row0 + r] / g.top_k);
        else src = (size_t)(tile.row0 + r);
        a_ptr[i] = g.A + src * t.row_bytes + t.kbase + (cbyte ^ (wave & 1) * 16);
    }
    const uint32_t a_lds = __builtin_amdgcn_readfirstlane(lds_addr_of(smem)) + wave * 1024;
    const uint32_t w_lds = a_lds + TL::W_RING + wave * ((W_PASS - 1) * 1024);

    f32x16 acc[NBT][WB];
#pragma unroll
    for (int m = 0; m < NBT; ++m)
#pragma unroll
        for (int b = 0; b < WB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[m][b][v] = 0.f;

    // where the next token / weight copies read and write: byte offset along K (wraps around), LDS address
    const int k_end = nk * GM_STEP_BYTES;
    int ka = t.koff * GM_STEP_BYTES, kw = ka;
    uint32_t a_dst = a_lds, w_dst = w_lds;
    auto advance = [&](int &k) __attribute__((always_inline)) { k += GM_STEP_BYTES; k = k == k_end ? 0 : k; };
    auto copy_token = [&](int i) __attribute__((always_inline)) {
        copy16_to_lds<false>(a_ptr[i] + ka, a_dst + i * (NW * 1024));
        if (i == A_PASS - 1) { advance(ka); a_dst = a_dst == a_lds ? a_lds + TL::A_STAGE : a_lds; }
    };
    auto copy_weight = [&](int i) __attribute__((always_inline)) {
        copy16_to_lds_at<false>(w_base + kw, w_off[i], w_dst + i * 1024);
        if (i == W_PASS - 1) { advance(kw); w_dst = w_dst == w_lds + 2 * TL::W_STAGE ? w_lds : w_dst + TL::W_STAGE; }
    };
    auto copy_tokens = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < A_PASS; ++i) copy_token(i);
    };
    auto copy_weights = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < W_PASS; ++i) copy_weight(i);
    };
    // lane (l32, lh) of a fragment holds chunk 2*kk + lh of row l32; the chunks of kk 0..3 are those of
    // kk = 0 with bits 1 and 2 of the chunk number flipped
    const int chunk = (lh ^ (l32 & 7) ^ (l32 >> 3 & 1)) << 4;
    int to = (TB0 * 32 + l32) * 128 + chunk, wo = TL::W_RING + (wn * 64 + l32) * 128 + chunk;
    bf16x8 wf[2][WB], tf[PF];
#define MOE_TOK(to_, q_) (*reinterpret_cast<const bf16x8 *>(smem + ((to_) ^ (((q_) / NBT) * 32)) + ((q_) % NBT) * 4096))
#define MOE_WGT(wo_, kk_, b_) (*reinterpret_cast<const bf16x8 *>(smem + ((wo_) ^ ((kk_) * 32)) + (b_) * 4096))

    copy_tokens();                                            // stage 0
    copy_weights();
    if (nk > 1) {                                             // stage 1
        copy_weights();
#pragma unroll
        for (int c = 0; c < NPRE; ++c) copy_token(c);
    }
    if (nk > 1) MOE_WAIT_VMCNT(W_PASS + NPRE);
    else MOE_WAIT_VMCNT(0);
    asm volatile("s_barrier" ::: "memory");
#pragma unroll
    for (int b = 0; b < WB; ++b) wf[0][b] = MOE_WGT(wo, 0, b);
#pragma unroll
    for (int q = 0; q < PF; ++q) tf[q] = MOE_TOK(to, q);
    __builtin_amdgcn_sched_barrier(0);

    int ws = 0;                                               // weight slot of this step
    // Step s issues the token copies of step s+1 and the weight copies of step s+2, spread over its groups.
    // LEFT: steps after this one, 0, 1 or (2) more
    auto step = [&](auto left_) __attribute__((always_inline)) {
        constexpr int LEFT = decltype(left_)::value;
        const int to_next = to ^ TL::A_STAGE;
        ws = ws == 2 ? 0 : ws + 1;
        const int wo_next = ws == 0 ? wo - 2 * TL::W_STAGE : wo + TL::W_STAGE;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int kk = q / NBT, m = q % NBT;
#pragma unroll
            for (int b = 0; b < WB; ++b)
                acc[m][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[kk & 1][b], tf[q % PF], acc[m][b], 0, 0, 0);
            if (q + PF < NQ) tf[q % PF] = MOE_TOK(to, q + PF);
            if (m == 0 && kk + 1 < NKK) {                     // the next 16 columns' weights
#pragma unroll
                for (int b = 0; b < WB; ++b) wf[(kk + 1) & 1][b] = MOE_WGT(wo, kk + 1, b);
            }
            // (issued in one go the copies would hold the wavefront up until the memory pipeline has taken
            // them all); the first of step s+1's token copies follow this step's meeting
            if (q <= QB) {
#pragma unroll
                for (int c = NPRE + q * CPG; c < NPRE + (q + 1) * CPG; ++c) {
                    if (c < A_PASS) {
                        if (LEFT >= 1) copy_token(c);
                    } else if (c < A_PASS + W_PASS) {
                        if (LEFT >= 2) copy_weight(c - A_PASS);
                    }
                }
            }
            if (LEFT >= 1) {
                if (q == QB) {
                    // every fragment of this stage has been requested: once they are here, and the next
                    // stage has landed, all wavefronts meet; then this stage may be overwritten
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                    if (LEFT >= 2) MOE_WAIT_VMCNT(W_PASS);
                    else MOE_WAIT_VMCNT(0);
                    asm volatile("s_barrier" ::: "memory");
#pragma unroll
                    for (int b = 0; b < WB; ++b) wf[0][b] = MOE_WGT(wo_next, 0, b);
#pragma unroll
                    for (int j = 0; j <= QB - (NQ - PF); ++j) tf[j] = MOE_TOK(to_next, j);
                }
                if (q > QB) tf[q - (NQ - PF)] = MOE_TOK(to_next, q - (NQ - PF));
                if (LEFT >= 2 && q >= QB) {
#pragma unroll
                    for (int c = (q - QB) * CPG; c < (q - QB + 1) * CPG && c < NPRE; ++c) copy_token(c);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        to = to_next;
        wo = wo_next;
    };
    for (int s = 0; s + 2 < nk; ++s) step(std::integral_constant<int, 2>{});
    if (nk > 1) step(std::integral_constant<int, 1>{});
    step(std::integral_constant<int, 0>{});
    MOE_WAIT_VMCNT(0);                                        // (nothing is in flight; cheap insurance for the LDS reuse below)
#undef MOE_TOK
#undef MOE_WGT

    // ---- epilogue: the output tile is staged in LDS and leaves as whole rows (see gemm_tile).  Lane
    // (l32, lh) holds, for token l32 of a block, weight rows 8*j + 4*lh .. +3 in registers 4*j .. 4*j+3.
    const int wcol = wn * (SH::COLS / 4);                     // this wavefront's first column inside the slab
    const int tid = t.tid;
    if constexpr (SH::SPLITK) {
        constexpr int NBT0 = (TB + 1) / 2;                    // blocks of the first half of the tile's rows
        constexpr int ROW_B = SH::COLS * 4, CPR = ROW_B / 16;
        constexpr int PARTS = (2 * NBT0 * 32 * ROW_B + TL::LDS_BYTES - 1) / TL::LDS_BYTES;
        constexpr int NBP = (NBT0 + PARTS - 1) / PARTS;       // row blocks of each half that leave together
        static_assert(2 * NBP * 32 * ROW_B <= TL::LDS_BYTES, "a part of the output tile must fit the LDS of the rings");
        auto stage_at = [&](int r, int byte) __attribute__((always_inline)) {
            return smem + r * ROW_B + ((((byte >> 4) ^ ((r & (CPR / 2 - 1)) << 1))) << 4) + (byte & 15);
        };
        unsigned char *const part_out = g.out + (size_t)t.kh * g.split_stride;
        const size_t out_pitch = (size_t)n_out * 4;
#pragma unroll
        for (int part = 0; part < PARTS; ++part) {
            const int m0 = part * NBP;
            __syncthreads();
#pragma unroll
            for (int m = m0; m < m0 + NBP && m < NBT; ++m) {
                const int r = ((TB0 ? NBP : 0) + m - m0) * 32 + l32;
#pragma unroll
                for (int b = 0; b < WB; ++b)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        *reinterpret_cast<f32x4 *>(stage_at(r, (wcol + b * 32 + j * 8 + lh * 4) * 4)) =
                            f32x4{acc[m][b][4 * j], acc[m][b][4 * j + 1], acc[m][b][4 * j + 2], acc[m][b][4 * j + 3]};
            }
            __syncthreads();
            for (int c = tid; c < 2 * NBP * 32 * CPR; c += SH::THREADS) {
                const int r = c / CPR, ch = c % CPR;
                const int half = r / (NBP * 32), in_half = m0 * 32 + r % (NBP * 32);
                const int trow = half * (NBT0 * 32) + in_half;
                const int col = ct * SH::COLS + ch * 4;
                if ((half || in_half < NBT0 * 32) && trow < rows && col < n_out) {
                    const u32x4 v = *reinterpret_cast<const u32x4 *>(stage_at(r, ch * 16));
                    u32x4 *dst = reinterpret_cast<u32x4 *>(part_out + (size_t)(tile.row0 + trow) * out_pitch + (size_t)col * 4);
                    if (g.nt_out) __builtin_nontemporal_store(v, dst);
                    else *dst = v;
                }
            }
        }
    } else {
        constexpr int ROW_B = SH::COLS * 2, CPR = ROW_B / 16;
        static_assert(TB * 32 * ROW_B <= TL::LDS_BYTES, "output tile must fit the LDS of the rings");
        auto stage_at = [&](int r, int byte) __attribute__((always_inline)) {
            return smem + r * ROW_B + ((((byte >> 4) ^ ((r & (CPR / 2 - 1)) << 1))) << 4) + (byte & 15);
        };
        __syncthreads();
#pragma unroll
        for (int m = 0; m < NBT; ++m) {
            const int r = (TB0 + m) * 32 + l32;
            if constexpr (SWIGLU) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float a[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const float gt = acc[m][0][4 * j + v], up = acc[m][1][4 * j + v];
                        a[v] = gt / (1.f + __expf(-gt)) * up;
                    }
                    uint2 o;
                    o.x = pack_bf16x2(a[0], a[1]);
                    o.y = pack_bf16x2(a[2], a[3]);
                    *reinterpret_cast<uint2 *>(stage_at(r, (wcol + j * 8 + lh * 4) * 2)) = o;
                }
            } else {
#pragma unroll
                for (int b = 0; b < WB; ++b)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        uint2 o;
                        o.x = pack_bf16x2(acc[m][b][4 * j], acc[m][b][4 * j + 1]);
                        o.y = pack_bf16x2(acc[m][b][4 * j + 2], acc[m][b][4 * j + 3]);
                        *reinterpret_cast<uint2 *>(stage_at(r, (wcol + b * 32 + j * 8 + lh * 4) * 2)) = o;
                    }
            }
        }
        __syncthreads();
        const size_t out_pitch = (size_t)n_out * 2;
        for (int c = tid; c < rows * CPR; c += SH::THREADS) {
            const int r = c / CPR, ch = c % CPR;
            const int col = ct * SH::COLS + ch * 8;
            if (col < n_out) {
                const u32x4 v = *reinterpret_cast<const u32x4 *>(stage_at(r, ch * 16));
                u32x4 *dst = reinterpret_cast<u32x4 *>(g.out + (size_t)(tile.row0 + r) * out_pitch + (size_t)col * 2);
                if (g.nt_out) __builtin_nontemporal_store(v, dst);
                else *dst = v;
            }
        }
    }
}

// TB: 32-row blocks of the tile.  The first four wavefronts take the first (TB+1)/2 of them, the others the
// rest: a compute unit's four matrix pipes each hold one wavefront of either half.
template <class SH, int TB>
__device__ __forceinline__ void gemm_tile_tall16(const GemmArgs &g, const Item &item, unsigned char *smem)
{
    constexpr int ES = 2;
    int tid_opaque = threadIdx.x;                             // (see gemm_tile)
    asm volatile("" : "+v"(tid_opaque));
    const size_t row_bytes = (size_t)g.K * ES;
    const int ct = SH::SPLITK ? item.ct >> 1 : item.ct, kh = SH::SPLITK ? item.ct & 1 : 0;
    const int nk = (int)(row_bytes / GM_STEP_BYTES) / (SH::SPLITK ? 2 : 1);
    // Workgroups that share weight and token lines through L2 start at the same column, experts (XCDs) at different ones:
    // with a start per workgroup the Mixtral gate/up launch of 4096 tokens fetched 7.9 GB, with this 4.9.
    const int koff = (int)((long)(item.tile.expert * 5 % g.k_groups) * nk / g.k_groups);
    const int wave = __builtin_amdgcn_readfirstlane(tid_opaque >> 6);
    const Tall16Args t{g, item.tile, smem, tid_opaque, tid_opaque & 63, wave, ct, kh, nk, koff,
                         row_bytes, (size_t)kh * nk * GM_STEP_BYTES};
    constexpr int NBT0 = (TB + 1) / 2, NBT1 = TB / 2;
    if (wave < 4) tall16_wave<SH, TB, NBT0, 0>(t);
    else tall16_wave<SH, TB, NBT1, NBT0>(t);
}

}  // namespace
}  // namespace moe

// Convolution with the lowering fused into the matrix product (gfx950, bf16, stride 1).
//
// The lowered matrix D-hat repeats every input element kh*kw times (App. C: the replication factor of
// the lowering phase), and the explicit path moves it through HBM several times per training step.
// This kernel computes the same product  Y-hat[F x M] = K-hat[F x K] * D-hat[K x M]  without D-hat ever
// existing in memory: a workgroup that owns 256 consecutive columns m = (n, oy, ox) keeps the zero-padded
// input pixels those columns touch in LDS, one 32-channel chunk at a time, and reads its MFMA operand
// straight out of that patch -- entry ((c, ky, kx), m) of D-hat is the patch pixel (oy + ky, ox + kx) of
// channel c, so a window tap is a constant LDS offset.  The reduction runs over (chunk, tap, channel in
// chunk); a sum does not care about the order of its terms, and the weights are repacked to match.
//
// The data gradient of a stride-1 layer is the same computation with the roles of the two channel
// counts exchanged, the window flipped and padding k - 1 - p (the col2im sum, written as a gather), so
// it runs on the same kernel and needs neither dD-hat nor a scatter step.
//
// LDS layout: patch[g][pixel] and atile[tap][g][row] of 16-byte packs, pack g holding channels
// 8g .. 8g+7 of the chunk, so a fragment is one 16-byte read per lane and consecutive lanes (consecutive
// pixels or rows) read consecutive packs.  Pixels are transposed from the input's [channel][pixel]
// order in registers on their way into LDS (8 channels x 7 or 8 pixels per thread, see pick_piece).  Padding pixels are
// zeroed once: the patch layout is the same for every chunk, and loads only ever write real pixels.
//
// Schedule: the weights of up to TG window taps are staged in LDS together, in one of two buffers, so a
// workgroup runs TG taps (TG x 8 MFMAs per wavefront) between barriers.  While it does, the next group's
// weights and -- during a chunk's first group -- the next chunk's pixels are in flight into registers.  The
// weights go to the other buffer before the group's last tap (every wavefront left that buffer before the last
// barrier), so those stores run under the other wavefronts' MFMAs and one barrier per group publishes them;
// only the pixels, once per chunk, need a barrier of their own before they overwrite the patch.
#include <cstring>
#include <type_traits>

#include "common.h"
#include "fused_geom.h"
#include "mma_epilogue.h"
#include "pack_jobs.h"

namespace omni {
namespace fused {

// Columns (output positions) per workgroup and the patch capacity in pixels that goes with them.  The wide
// tile gives each wavefront 64 x 128 results: 6 instead of 8 LDS fragment reads per 8 MFMAs, and LDS
// bandwidth is what caps this kernel.
constexpr int BN_SMALL = 128, PATCH_SMALL = 576;  // with 64 rows and 4 wavefronts: two workgroups per compute unit
constexpr int BN_NARROW = 256, PATCH_NARROW = 672;
constexpr int BN_MID = 384, PATCH_MID = 960;
constexpr int BN_WIDE = 512, PATCH_WIDE = 1040;
constexpr int TG = 5;            // window taps whose weights are staged in LDS together (two such buffers)

static int g_fused_bn = 0, g_fused_bm = 0, g_fused_bare_pitch = 0, g_fused_whole = 0;  // omni_tuning_set(OMNI_TUNE_FUSED_*): sweeps and tests only

// Patch pixels of pieces of 8 (SWZ) are stored at swz(pixel): a loader thread writes 8 consecutive pixels and its neighbour the
// next 8, so without the permutation every lane of a store would fall on the same two bank groups.  The permutation stays
// inside aligned blocks of 8, so a run of consecutive pixels read by consecutive lanes still covers all banks.
template <bool SWZ> __device__ __forceinline__ int swz(int pix) { return SWZ ? pix ^ ((pix >> 4) & 7) : pix; }

// Epi: FwdEpilogue<bf16_t> (bias, ReLU, rounding, store into Y), or PartialEpilogue when few column tiles
// exist (small batches): the reduction's chunks are then split over `g.splits` workgroups per tile, each
// leaving its raw fp32 sums in a slice [F][M] of the scratch, which reduce_store_kernel adds in split order
// and hands to the forward epilogue.
// RIN: the input is read with the strides g.sn, g.sc (its rows form) instead of as the dense tensor.
// SWZ: loader pieces of 8 elements, permuted (of the rows form they are not); else of g.piece, which is 7 for the dense tensor.
template <int BM, int WM, int WN, int BN, int PATCH_PIX, typename Epi, bool RIN = false, bool SWZ = false>
__global__ __launch_bounds__(64 * WM * WN, 2) void fused_conv_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ Wt,
                                                        Geom g, Epi epi)
{
    constexpr int NT = 64 * WM * WN;
    static_assert(BM * NG <= NT, "at most one 16-byte piece of a tap's weight tile per thread");
    constexpr int TI = BM / WM / 32, TJ = BN / WN / 32;
    constexpr int LA = BM + 1;
    __shared__ uint4 patch[NG * PATCH_PIX];
    __shared__ uint4 atile[2 * TG * NG * LA];
    __shared__ float lds_add[BM];
    __shared__ int slot_so[MAX_SLOTS], slot_ra[MAX_SLOTS], slot_p0[MAX_SLOTS], slot_ya[MAX_SLOTS], slot_len[MAX_SLOTS];
    __shared__ int total_pieces;

    const int xcd = blockIdx.x % 8, slot_id = blockIdx.x / 8;
    const int item = xcd * g.per_xcd + slot_id;  // contiguous ranges of tiles per XCD, row tiles fastest
    if (item >= g.n_items) return;
    const int n_tiles = g.tiles_f * g.tiles_m;
    const int z = item / n_tiles, tile_id = item - z * n_tiles;   // splits of one tile are far apart in time
    const int chunk_lo = z * g.chunks_per_split;
    const int chunk_hi = chunk_lo + g.chunks_per_split < g.n_chunks ? chunk_lo + g.chunks_per_split : g.n_chunks;
    const int tm = tile_id / g.tiles_f, tf = tile_id - tm * g.tiles_f;
    const int row0 = tf * BM, col0 = tm * BN;
    const int m_last = (col0 + BN < g.M ? col0 + BN : g.M) - 1;
    const int n0 = (int)g.div_HoWo.div((uint32_t)col0);
    const int nslots = (int)g.div_HoWo.div((uint32_t)m_last) - n0 + 1;

    const int tid = threadIdx.x;
    const int lane = tid % 64, wave = tid / 64;
    const int wm = wave / WN, wn = wave % WN;
    const int li = lane % 32, h = lane / 32;

    // elements of a loader task; constants wherever they can be (a division in thread 0's loop is time that all others wait)
    const bool sevens = !SWZ && (!RIN || g.piece == 7);
    const int piece = sevens ? 7 : 8;
    if (tid == 0) {
        int so = 0, p0 = 0;
        for (int i = 0; i < nslots; ++i) {
            SlotSpan s = slot_span(g, col0, m_last, n0 + i);
            slot_so[i] = so, slot_ra[i] = s.ra, slot_p0[i] = p0, slot_ya[i] = s.ya, slot_len[i] = s.len;
            so += s.nrows;
            p0 += sevens ? (s.len + 6) / 7 : (s.len + 7) / 8;
        }
        total_pieces = p0;
    }
    __syncthreads();

    // patch pixel of each of this lane's columns at tap (0, 0)
    int pp0[TJ];
#pragma unroll
    for (int u = 0; u < TJ; ++u) {
        int m = col0 + wn * (BN / WN) + 32 * u + li;
        m = m < g.M ? m : g.M - 1;
        uint32_t n, q, oy, ox;
        g.div_HoWo.divmod((uint32_t)m, n, q);
        g.div_Wo.divmod(q, oy, ox);
        int i = (int)n - n0;
        pp0[u] = (slot_so[i] + (int)oy - slot_ra[i]) * g.Wp + (int)ox;
    }

    // This thread's share of a chunk: 8 channels (pack tg) x 7 or 8 (piece) consecutive elements of one image's rows.
    const int PT = total_pieces;
    const bool has_task = tid < NG * PT;
    uint32_t goff = 0;                        // byte offset of the task's first element in chunk 0
    uint32_t l01 = NO_PIX | (NO_PIX << 16), l23 = l01, l45 = l01, l67 = l01;  // patch index of each element
    if (has_task) {
        int tg = tid / PT, jj = tid - tg * PT;
        int i = nslots - 1;
        while (i > 0 && jj < slot_p0[i]) --i;
        int ea = slot_ya[i] * g.W, eb = ea + slot_len[i];
        int e0 = ea + piece * (jj - slot_p0[i]);
        e0 = e0 < g.HW - piece ? e0 : g.HW - piece;  // stay inside the plane: the overlap rewrites equal values
        if constexpr (RIN) goff = ((uint32_t)(n0 + i) * g.sn + (uint32_t)(8 * tg) * g.sc + (uint32_t)e0) * 2u;
        else goff = ((uint32_t)((n0 + i) * g.C + 8 * tg) * (uint32_t)g.HW + (uint32_t)e0) * 2u;
        uint32_t l[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            int flat = e0 + e;
            uint32_t y, x;
            g.div_W.divmod((uint32_t)flat, y, x);
            int pp = (slot_so[i] + (int)y + g.ph - slot_ra[i]) * g.Wp + (int)x + g.pw;
            l[e] = (flat >= ea && flat < eb && e < piece) ? (uint32_t)(tg * PATCH_PIX + swz<SWZ>(pp)) : NO_PIX;
        }
        l01 = l[0] | (l[1] << 16), l23 = l[2] | (l[3] << 16), l45 = l[4] | (l[5] << 16), l67 = l[6] | (l[7] << 16);
    }

    u32x4 r0, r1, r2, r3, r4, r5, r6, r7;  // 8 channels x 8 elements
    const char *xb = reinterpret_cast<const char *>(X);
    const uint32_t plane_b = (RIN ? g.sc : (uint32_t)g.HW) * 2u, chunk_b = plane_b * CH;
    // Pieces of 7: every channel's load starts at the multiple of 4 bytes at or before its first element.  Two planes, and a
    // chunk's, are a multiple of 4 bytes, so whether it starts one element early is the same for every second channel.
    const uint32_t goff_e = sevens ? goff & ~3u : goff, goff_o = sevens ? (goff + plane_b) & ~3u : goff + plane_b;
    const uint32_t shift_e = (goff - goff_e) * 8u, shift_o = (goff + plane_b - goff_o) * 8u;
    auto issue_patch = [&](int chunk) {
        const char *p = xb + (goff_e + (uint32_t)chunk * chunk_b);  // threads without a task read a valid address too
        const char *q = SWZ ? p + plane_b : xb + (goff_o + (uint32_t)chunk * chunk_b);
        __builtin_memcpy(&r0, p, 16);
        __builtin_memcpy(&r1, q, 16);
        __builtin_memcpy(&r2, p + 2 * plane_b, 16);
        __builtin_memcpy(&r3, q + 2 * plane_b, 16);
        __builtin_memcpy(&r4, p + 4 * plane_b, 16);
        __builtin_memcpy(&r5, q + 4 * plane_b, 16);
        __builtin_memcpy(&r6, p + 6 * plane_b, 16);
        __builtin_memcpy(&r7, q + 6 * plane_b, 16);
    };
    auto unshift = [](u32x4 &r, uint32_t shift) {
        r = u32x4{__builtin_amdgcn_alignbit(r[1], r[0], shift), __builtin_amdgcn_alignbit(r[2], r[1], shift),
                  __builtin_amdgcn_alignbit(r[3], r[2], shift), r[3] >> shift};
    };
    auto commit_patch = [&]() {
        if (sevens) {
            unshift(r0, shift_e), unshift(r2, shift_e), unshift(r4, shift_e), unshift(r6, shift_e);
            unshift(r1, shift_o), unshift(r3, shift_o), unshift(r5, shift_o), unshift(r7, shift_o);
        }
        u32x4 *dst = reinterpret_cast<u32x4 *>(patch);
        uint32_t l;
        // element e of the 8 x 8 block as one pack: the 8 channels of that pixel
        l = l01 & 0xffffu; if (l != NO_PIX) dst[l] = u32x4{lo16(r0[0], r1[0]), lo16(r2[0], r3[0]), lo16(r4[0], r5[0]), lo16(r6[0], r7[0])};
        l = l01 >> 16;     if (l != NO_PIX) dst[l] = u32x4{hi16(r0[0], r1[0]), hi16(r2[0], r3[0]), hi16(r4[0], r5[0]), hi16(r6[0], r7[0])};
        l = l23 & 0xffffu; if (l != NO_PIX) dst[l] = u32x4{lo16(r0[1], r1[1]), lo16(r2[1], r3[1]), lo16(r4[1], r5[1]), lo16(r6[1], r7[1])};
        l = l23 >> 16;     if (l != NO_PIX) dst[l] = u32x4{hi16(r0[1], r1[1]), hi16(r2[1], r3[1]), hi16(r4[1], r5[1]), hi16(r6[1], r7[1])};
        l = l45 & 0xffffu; if (l != NO_PIX) dst[l] = u32x4{lo16(r0[2], r1[2]), lo16(r2[2], r3[2]), lo16(r4[2], r5[2]), lo16(r6[2], r7[2])};
        l = l45 >> 16;     if (l != NO_PIX) dst[l] = u32x4{hi16(r0[2], r1[2]), hi16(r2[2], r3[2]), hi16(r4[2], r5[2]), hi16(r6[2], r7[2])};
        l = l67 & 0xffffu; if (l != NO_PIX) dst[l] = u32x4{lo16(r0[3], r1[3]), lo16(r2[3], r3[3]), lo16(r4[3], r5[3]), lo16(r6[3], r7[3])};
        l = l67 >> 16;     if (l != NO_PIX) dst[l] = u32x4{hi16(r0[3], r1[3]), hi16(r2[3], r3[3]), hi16(r4[3], r5[3]), hi16(r6[3], r7[3])};
    };

    // The weight tile of reduction step st = chunk * KK + tap is [g][Fp] packs, contiguous per g; this
    // thread moves pack (tid / BM, row0 + tid % BM) of each of a group's TG tiles.  Requests are
    // unconditional: steps past the group's (or the reduction's) end repeat a valid tile that nobody reads.
    static_assert(TG <= 9, "named staging registers below");
    u32x4 a0, a1, a2, a3, a4, a5, a6, a7, a8;  // named so that each stays a register
    auto areg = [&](auto q) -> u32x4 & {
        constexpr int Q = decltype(q)::value;
        if constexpr (Q == 0) return a0; else if constexpr (Q == 1) return a1; else if constexpr (Q == 2) return a2;
        else if constexpr (Q == 3) return a3; else if constexpr (Q == 4) return a4; else if constexpr (Q == 5) return a5;
        else if constexpr (Q == 6) return a6; else if constexpr (Q == 7) return a7; else return a8;
    };
    const int KK = g.KK, n_steps = g.n_chunks * KK;
    const bool has_piece = tid < BM * NG;            // a 96-row tile has fewer pieces than threads
    const int wtid = has_piece ? tid : BM * NG - 1;  // the others repeat the last one's (valid) requests
    const u32x4 *wt_tile = reinterpret_cast<const u32x4 *>(Wt) + row0;  // wave-uniform
    const uint32_t wt_off = (uint32_t)((wtid / BM) * g.Fp + wtid % BM) * 16u;
    const u32x4 *wt = wt_tile + (wtid / BM) * g.Fp + wtid % BM;
    const int step_stride = NG * g.Fp;  // packs from one step's tile to the next
    u32x4 *const at = reinterpret_cast<u32x4 *>(atile) + (wtid / BM) * LA + wtid % BM;
    // Tiles whose pieces are one per thread (BM * NG == NT, BM a multiple of 64) go from global memory straight
    // into LDS: a wavefront's 64 pieces are 64 consecutive packs of one channel pack, in memory and in the tile,
    // so one global-to-LDS load per tap and wavefront (LDS address = a wave-uniform base + lane * 16) replaces a
    // load into registers, the registers themselves and an LDS store.  The loads are asynchronous: they are waited
    // for (memory counter at zero) before the barrier that publishes the buffer.
    constexpr bool DMA = BM * NG == NT && BM % 64 == 0;
    u32x4 *const at_wave = reinterpret_cast<u32x4 *>(atile) + __builtin_amdgcn_readfirstlane((wave * 64 / BM) * LA + (wave * 64) % BM);
    auto issue_a = [&](int st0, int buf) {
        static_for<0, TG>([&](auto q) {
            int st = st0 + decltype(q)::value;
            st = st < n_steps ? st : n_steps - 1;
            if constexpr (DMA)
                lds_dma16(wt_tile + (int64_t)st * step_stride, wt_off, at_wave + (buf * TG + decltype(q)::value) * (NG * LA));
            else
                areg(q) = wt[st * step_stride];
        });
    };
    auto commit_a = [&](int buf) {
        if constexpr (!DMA)
            if (has_piece)
                static_for<0, TG>([&](auto q) { at[(buf * TG + decltype(q)::value) * (NG * LA)] = areg(q); });
    };
    auto wait_a = [&]() {
        if constexpr (DMA) lds_dma_wait();
    };

    f32x16 acc[TI][TJ];
#pragma unroll
    for (int t = 0; t < TI; ++t)
#pragma unroll
        for (int u = 0; u < TJ; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][u][v] = 0.f;

    // A tap is two slabs of MFMAs (channel packs 0, 1 and 2, 3 of the chunk).  The fragments of a slab are read
    // from LDS one slab ahead, into the other of two register sets, so that a wavefront's LDS latency runs
    // under its own MFMAs and not only under the other wavefront's.
    uint4 fa0[TI], fb0[TJ], fa1[TI], fb1[TJ];
    int pix[TJ];
    auto set_pix = [&](int tapoff) {
#pragma unroll
        for (int u = 0; u < TJ; ++u) pix[u] = swz<SWZ>(pp0[u] + tapoff);
    };
    auto load_frag = [&](uint4 (&fa)[TI], uint4 (&fb)[TJ], int buf, int slot, int s2) {
        const int g2 = 2 * s2 + h;
        const uint4 *pa = atile + (buf * TG + slot) * (NG * LA) + wm * (BM / WM) + li + g2 * LA;
#pragma unroll
        for (int t = 0; t < TI; ++t) fa[t] = pa[32 * t];
#pragma unroll
        for (int u = 0; u < TJ; ++u) fb[u] = patch[g2 * PATCH_PIX + pix[u]];
    };
    auto mma_frag = [&](const uint4 (&fa)[TI], const uint4 (&fb)[TJ]) {
#pragma unroll
        for (int t = 0; t < TI; ++t)
#pragma unroll
            for (int u = 0; u < TJ; ++u) Mma<bf16_t>::run(fa[t], fb[u], acc[t][u]);
    };

    // The first chunk's pixels and weights are requested before the patch is cleared, so that the clearing (the
    // padding stays zero for the whole kernel: loads only ever write real pixels) runs under their latency.
    issue_patch(chunk_lo);
    issue_a(chunk_lo * KK, 0);
    for (int i = tid; i < NG * PATCH_PIX; i += NT) patch[i] = make_uint4(0, 0, 0, 0);
    if constexpr (Epi::HAS_ROW_ADD)
        for (int i = tid; i < BM; i += NT) lds_add[i] = epi.row_add(row0 + i);
    __syncthreads();
    commit_patch();
    commit_a(0);
    wait_a();
    __syncthreads();
    int ky = 0, kx = 0, buf = 0;
    for (int chunk = chunk_lo; chunk < chunk_hi; ++chunk) {
        const bool more_chunks = chunk + 1 < chunk_hi;
        for (int t0 = 0; t0 < KK; t0 += TG) {
            const int nt = KK - t0 < TG ? KK - t0 : TG;
            const bool last_group = t0 + TG >= KK;
            issue_a(chunk * KK + t0 + nt, buf ^ 1);            // the next group (of this chunk or the next)
            if (t0 == 0 && more_chunks) issue_patch(chunk + 1);
            // The next group's weights go to the other buffer (free since the last barrier) before this
            // group's last tap, so that those stores run under the other wavefronts' MFMAs.
            set_pix(ky * g.Wp + kx);
            load_frag(fa0, fb0, buf, 0, 0);
            for (int t = 0; t < nt; ++t) {
                load_frag(fa1, fb1, buf, t, 1);
                if (t == nt - 1) commit_a(buf ^ 1);
                mma_frag(fa0, fb0);
                if (++kx == g.kw) kx = 0, ++ky;
                if (t + 1 < nt) {
                    set_pix(ky * g.Wp + kx);
                    load_frag(fa0, fb0, buf, t + 1, 0);
                }
                mma_frag(fa1, fb1);
            }
            if (last_group) ky = 0;
            if (last_group && more_chunks) {
                __syncthreads();  // every wavefront has read this chunk's pixels
                commit_patch();
            }
            wait_a();
            __syncthreads();      // this group's weights are free, the next group's (and chunk's pixels) are in LDS
            buf ^= 1;
        }
    }

    // every wavefront is past the loop's last barrier: the weight tiles become staging space
    constexpr int STRIP = 16 * staged_pitch(TJ);
    static_assert((NT / 64) * STRIP <= (int)sizeof(atile), "staging strips fit in the weight tiles");
    if constexpr (epilogue_is_masked<Epi>::value) {
        // the patch is free as well: [BM][WN] sums of what each wavefront stored per row, added in wavefront order
        float *wave_sums = reinterpret_cast<float *>(patch);
        static_assert(BM * WN * 4 <= (int)sizeof(patch), "row sums fit in the patch");
        store_tile_staged<TI, TJ, 16>(acc, row0 + wm * (BM / WM), col0 + wn * (BN / WN), lane, z, epi,
                                      reinterpret_cast<char *>(atile) + wave * STRIP, lds_add, row0, wave_sums, WN, wn);
        __syncthreads();
        if (epi.sums != nullptr && tid < BM && row0 + tid < g.F) {
            float total = 0.f;
#pragma unroll
            for (int w = 0; w < WN; ++w) total += wave_sums[tid * WN + w];
            epi.sums[(int64_t)(row0 + tid) * g.tiles_m + tm] = total;
        }
    } else {
        store_tile_staged<TI, TJ, 16>(acc, row0 + wm * (BM / WM), col0 + wn * (BN / WN), lane, z, epi,
                                      reinterpret_cast<char *>(atile) + wave * STRIP, lds_add, row0);
    }
}

// Weights [out][in][kh][kw] (forward) or [in][out][kh][kw] read flipped (data gradient) -> the kernel's
// order [chunk][tap][g][Fp][8]: pack (chunk, tap, g, row) = input channels chunk*32 + 8g .. +7 of output
// channel `row` at window tap `tap`; rows beyond F are zero.  One thread per pack (pack_one, pack_jobs.h); a launch
// carries a table of such jobs, block b belonging to the job whose block range holds it.
__global__ __launch_bounds__(256) void pack_jobs_kernel(PackJobTable t)
{
    int j = 0;
    while (j + 1 < t.n && (int64_t)blockIdx.x >= t.first_block[j + 1]) ++j;
    const int64_t p = ((int64_t)blockIdx.x - t.first_block[j]) * 256 + threadIdx.x;
    if (p < t.job[j].total) pack_one(t.job[j], p);
}

// What the column tiles of bn positions need at most: padded rows, and loader pieces of 8 and of 7 elements.  !fits: one
// touches too many images, or needs more rows or more pieces of 8 than allowed; then the scan ends there (a layer of large
// planes has thousands of tiles, and 1 x 64 x 4001 x 3999 is known not to fit after the first).
// (The tiles' positions inside an image repeat with period HoWo / gcd(bn, HoWo).)
struct TileExtent { bool fits; int rows, pieces8, pieces7; };
static TileExtent tile_extent(const Geom &g, int bn, int64_t most_rows, int most_pieces8)
{
    TileExtent t{false, 0, 0, 0};
    int tiles_m = (g.M + bn - 1) / bn;
    int a = bn, b = g.HoWo;
    while (b != 0) { int t = a % b; a = b, b = t; }
    int period = g.HoWo / a + 1;
    for (int tm = 0; tm < tiles_m && tm < period; ++tm) {
        int col0 = tm * bn, m_last = (col0 + bn < g.M ? col0 + bn : g.M) - 1;
        int n0 = col0 / g.HoWo, n1 = m_last / g.HoWo;
        if (n1 - n0 + 1 > MAX_SLOTS) return t;
        int rows = 0, pieces8 = 0, pieces7 = 0;
        for (int n = n0; n <= n1; ++n) {
            SlotSpan s = slot_span(g, col0, m_last, n);
            rows += s.nrows;
            pieces8 += (s.len + 7) / 8;
            pieces7 += (s.len + 6) / 7;
        }
        if (rows > most_rows || pieces8 > most_pieces8) return t;
        if (rows > t.rows) t.rows = rows;
        if (pieces8 > t.pieces8) t.pieces8 = pieces8;
        if (pieces7 > t.pieces7) t.pieces7 = pieces7;
    }
    t.fits = true;
    return t;
}

// Elements a loader task takes of each of its planes: 7 where the tasks fit that way, one per thread.  A 16-byte load from an
// address that is only 2-byte aligned costs a wavefront 65 cycles, from a multiple of 4 bytes 20: a task of 7 elements loads its
// 8 from the multiple of 4 bytes at or before its first and shifts them.  And the pixels then lie in LDS as they come, free of
// bank conflicts for the stores (neighbouring tasks 7 pixels apart) and for the fragment reads (consecutive pixels); pieces of 8
// needed a permutation that spread the stores but cost the reads nearly a second pass and an address computation per tap.
// 384 -> 384 channels, 13 x 13, 50 / 256 images: 44.7 / 110.6 -> 42.6 / 107.5 us; 256 -> 384, 50: 32.9 -> 29.5; data gradient
// of 96 -> 256, 27 x 27, window 5, 256 images: 252 -> 243.
// Windows of 1 x 1 on planes and rows of an even number of elements keep pieces of 8: those start at multiples of 4 bytes anyway,
// and with one tap per chunk the loads count for more than the permuted reads (416 -> 1760 channels, 34 x 32, 60 images, 224 us with
// pieces of 8, 247 with 7; 1 300 such layers 1.025 on average; windows of 3 on such planes 0.985, 1 x 1 on odd ones 0.9).
static int pick_piece(const Geom &g, const TileExtent &t, int threads)
{
    if (g.KK == 1 && g.HW % 2 == 0 && g.W % 2 == 0) return 8;
    return NG * t.pieces7 <= threads ? 7 : 8;
}

// The row pitch a Geom can have: the smallest with which its tiles' fragment reads are free of bank conflicts.
static int conflict_free_pitch(const Geom &g)
{
    int wp = g.W + 2 * g.pw;
    while ((wp - g.Wo) % 16 != 0) ++wp;
    return wp;
}

// The convolution as this kernel sees it, on the 128- and 96-row tiles; for the data gradient the layer's output
// gradient is the input and the window is flipped.
static bool plan_fused_geom(const ConvGeom &c, bool data_gradient, Geom *g)
{
    if (c.sh != 1 || c.sw != 1) return false;
    if (!data_gradient) {
        g->N = c.N, g->C = c.C, g->H = c.H, g->W = c.W, g->F = c.F, g->Ho = c.Ho, g->Wo = c.Wo;
        g->ph = c.ph, g->pw = c.pw;
    } else {
        g->N = c.N, g->C = c.F, g->H = c.Ho, g->W = c.Wo, g->F = c.C, g->Ho = c.H, g->Wo = c.W;
        g->ph = c.kh - 1 - c.ph, g->pw = c.kw - 1 - c.pw;
        if (g->ph < 0 || g->pw < 0) return false;
    }
    g->kh = c.kh, g->kw = c.kw;
    g->Wp = g->W + 2 * g->pw;  // replaced below by the pitch chosen with the tile
    g->config = -1, g->plane = 0, g->piece = 8, g->cols_fastest = 0;
    g->HW = g->H * g->W, g->HoWo = g->Ho * g->Wo, g->KK = c.kh * c.kw;
    g->sn = (uint32_t)g->C * (uint32_t)g->HW, g->sc = (uint32_t)g->HW;  // dense [N][C][H][W]; launch_fused_conv may replace them
    int64_t M = (int64_t)g->N * g->HoWo;
    if (g->C % CH != 0 || g->HW < 8 || M > 0x7fffffffll - 4096) return false;
    if ((double)g->N * g->C * g->HW * 2.0 >= 4.0e9 || (double)M * g->F * 2.0 >= 4.0e9) return false;
    g->M = (int32_t)M;
    g->n_chunks = g->C / CH;
    g->bm = 128;
    g->Fp = (int32_t)round_up(g->F, 128);
    g->tiles_f = g->Fp / 128;
    g->div_HoWo = FastDiv((uint32_t)g->HoWo);
    g->div_Wo = FastDiv((uint32_t)g->Wo);
    g->div_W = FastDiv((uint32_t)g->W);
    // Row pitch of the patch.  A fragment read takes its 64 lanes in four passes of 16 (lanes 0-3, 12-15, 20-27;
    // 4-11, 16-19, 28-31; the same of the upper half), each free of bank conflicts when its 16-byte slots differ
    // mod 16.  A lane's slot is the patch pixel of its output position, so with a pitch that equals the output
    // width mod 16 the slot is (position + constant) mod 16 also across row wraps, and consecutive positions never
    // collide; with the bare padded width every row wrap inside a pass shifts some lanes onto others' banks.
    const int wp_min = g->W + 2 * g->pw, wp_free = conflict_free_pitch(*g);
    // Few tiles (small batches): the reduction is cut into ranges of chunks so that about one workgroup per
    // compute unit exists; the ranges' fp32 sums are added in a fixed order afterwards.
    auto splits_for = [&](int64_t n_tiles, int64_t F_rows) {
        int splits = 1;
        if (n_tiles <= 128 && g->n_chunks >= 2 && (double)F_rows * g->M * 4.0 * 16.0 < 4.0e9) {
            int want = (int)(256 / n_tiles);
            splits = want < g->n_chunks ? want : g->n_chunks;
        }
        const int per = (g->n_chunks + splits - 1) / splits;
        return (g->n_chunks + per - 1) / per;
    };
    // Among the tiles that fit, the one with the least estimated time: rounds of the 256 compute units times the
    // tile's width times what a workgroup does per column -- the chunks of the reduction it walks plus its fixed
    // part (prologue and epilogue cost about as much as 14 window taps; a split reduction also writes fp32 partial
    // sums that are added afterwards) -- the narrower tiles a few per cent dearer per column (their weights are
    // staged for fewer columns, and they read more LDS fragments per MFMA).
    auto estimate = [&](int64_t tiles, int bn, double per_column, int64_t F_rows) {
        const int splits = splits_for(tiles, F_rows);
        const int per = (g->n_chunks + splits - 1) / splits;
        const double fixed = 14.0 / g->KK + (splits > 1 ? 0.5 : 0.0);
        return (double)((tiles * splits + 255) / 256) * bn * per_column * (per + fixed);
    };
    const int want = g_fused_bn == BN_SMALL ? 0 : g_fused_bn;  // tuning override: 256, 384 or 512 (0: choose)
    const struct { int bn, patch; double per_column; } tiles[3] = {
        {BN_WIDE, PATCH_WIDE, 1.0}, {BN_MID, PATCH_MID, 1.03}, {BN_NARROW, PATCH_NARROW, 1.06}};
    constexpr double CONFLICTS = 1.15;  // what the bare pitch costs per column (measured on the 27-wide layer)
    double best = 0.0;
    g->bn = 0;
    for (const auto &t : tiles) {
        if (want != 0 && want != t.bn) continue;
        const TileExtent e = tile_extent(*g, t.bn, t.patch / wp_min, 512 / NG);
        if (!e.fits) continue;
        const bool free_fits = !g_fused_bare_pitch && e.rows * wp_free <= t.patch;
        const double cost = estimate((int64_t)g->tiles_f * ((g->M + t.bn - 1) / t.bn), t.bn,
                                     t.per_column * (free_fits ? 1.0 : CONFLICTS), g->F);
        if (g->bn == 0 || cost < best) g->bn = t.bn, g->Wp = free_fits ? wp_free : wp_min, g->piece = pick_piece(*g, e, 512), best = cost;
    }
    // A layer of at most 64 filters takes a 96-row tile (8 wavefronts of 96 x 64 on 512 columns): three quarters
    // of the MFMAs for a few more fragment reads per MFMA.  (Measured: 48 filters 287 -> 192 us; with 96 filters
    // the two tiles take the same time, the kernel being bound by its LDS reads, so those keep the 128-row tile.)
    const int bm_want = g_fused_bm;  // tuning override: 128 keeps the 128-row tile, 96 forces the other up to 96 filters
    const int f_max = bm_want == 96 ? 96 : 64;
    if (g->F <= f_max && (bm_want == 0 || bm_want == 96) && (want == 0 || want == BN_WIDE)) {
        const TileExtent e = tile_extent(*g, BN_WIDE, PATCH_WIDE / wp_min, 512 / NG);
        if (e.fits) {
            const bool free_fits = !g_fused_bare_pitch && e.rows * wp_free <= PATCH_WIDE;
            const double cost = estimate((g->M + BN_WIDE - 1) / BN_WIDE, BN_WIDE, 0.8 * (free_fits ? 1.0 : CONFLICTS), g->F);
            if (g->bn == 0 || cost < best)
                g->bn = BN_WIDE, g->bm = 96, g->Fp = 96, g->tiles_f = 1, g->Wp = free_fits ? wp_free : wp_min, g->piece = pick_piece(*g, e, 512), best = cost;
        }
    }
    if (g->bn == 0) return false;
    g->tiles_m = (g->M + g->bn - 1) / g->bn;
    const int n_tiles = g->tiles_f * g->tiles_m;
    g->splits = splits_for(n_tiles, g->F);
    g->chunks_per_split = (g->n_chunks + g->splits - 1) / g->splits;
    g->splits = (g->n_chunks + g->chunks_per_split - 1) / g->chunks_per_split;
    g->n_items = n_tiles * g->splits;
    g->per_xcd = (g->n_items + 7) / 8;
    return true;
}

// Estimated time of a planned product in microseconds, the sum of the splits included: a fixed part, and per round of
// workgroups its own fixed part, the chunks' pixels and the taps.  Fitted to 3 700 measurements (19 layers of 32 to 384
// channels, planes of 8 x 8 to 32 x 32, windows of 1, 3 and 5, 1 to 256 images, every tile and 1 to 12 splits; mean
// deviation 6 %).  It is used beyond those ranges too: over 2 000 random layers of 32 to 1 024 channels, planes of 5 x 5 to
// 80 x 80 and windows of 1 to 11 a forward pass took at most 2 %, a data gradient 4 % longer than on the larger tiles alone.
// A tap of the small tile takes 0.14 us on a compute unit of its own and 0.27 beside another workgroup; a split costs its
// fp32 sums' way through memory and a launch.
static double estimated_us(const Geom &g)
{
    const double taps = (double)g.chunks_per_split * g.KK;
    const double sums = g.splits > 1 ? 1.0 : 0.0, mb = sums * (double)g.splits * g.F * g.M * 4e-6;
    if (g.bm == 64) {
        const int rounds = (g.n_items + 511) / 512;
        const double tap = rounds > 1 ? 0.22 : g.n_items > 256 ? 0.27 : 0.14;
        return 5.2 + 1.4 * (rounds - 1) + rounds * (1.0 * g.chunks_per_split + tap * taps) + 1.95 * sums + 0.325 * mb;
    }
    const int rounds = (g.n_items + 255) / 256;
    if (g.bn == BN_NARROW) return 5.6 + rounds * (0.4 + 1.3 * g.chunks_per_split + 0.336 * taps) + 1.95 * sums + 0.363 * mb;
    if (g.bn == BN_MID) return 7.0 + rounds * (2.1 + 1.4 * g.chunks_per_split + 0.477 * taps) + 1.1 * sums + 0.326 * mb;
    return 7.0 + rounds * (3.0 + 1.2 * g.chunks_per_split + (g.bm == 96 ? 0.42 : 0.611) * taps) + 0.65 * sums + 0.324 * mb;
}

// The same product on 64 x 128 tiles of four wavefronts: four times the workgroups of the next larger tile, two of them
// on a compute unit, so that a small batch fills the chip with fewer splits and fewer fp32 sums to write and add (384
// filters, 256 channels, 13 x 13: 16 images 26.5 -> 23 us, 50 images 40 -> 33, one image 13.1 -> 9.8; 32 channels, 16 x 16,
// window 5, 100 images 14.7 -> 9.9).  A large product keeps the wide tiles, which read fewer LDS fragments per MFMA (the
// first of these layers at 100 images: 60 us here, 43 there).  false: a column tile does not fit.
static bool plan_small_tile(const Geom &base, Geom *out)
{
    Geom g = base;
    g.bn = BN_SMALL, g.bm = 64;
    g.tiles_f = (g.F + 63) / 64, g.tiles_m = (g.M + BN_SMALL - 1) / BN_SMALL;  // Fp, the packed weights' order, stays
    g.Wp = conflict_free_pitch(g);
    const int wp_min = g.W + 2 * g.pw;
    const TileExtent e = tile_extent(g, BN_SMALL, PATCH_SMALL / wp_min, 256 / NG);
    if (!e.fits) return false;
    if (g_fused_bare_pitch || e.rows * g.Wp > PATCH_SMALL) g.Wp = wp_min;
    g.piece = pick_piece(g, e, 256);
    const int n_tiles = g.tiles_f * g.tiles_m;
    // A layer whose larger tiles fit the library's own scratch has to fit it here too.
    const double packed = (double)g.n_chunks * g.KK * NG * g.Fp * 16.0, slice = (double)g.F * g.M * 4.0;
    const double base_sums = base.splits > 1 ? base.splits * slice : 0.0, room = (double)OMNI_STATIC_SCRATCH_BYTES - 256.0 - packed;
    const double most_sums = base_sums > room ? base_sums : room;
    bool found = false;
    double least = 0.0;
    for (int per = g.n_chunks; per >= 1; --per) {
        const int splits = (g.n_chunks + per - 1) / per;
        if (splits > 1 && (base.whole || (int64_t)n_tiles * splits > 1024 || splits * slice > most_sums)) break;
        g.splits = splits, g.chunks_per_split = per, g.n_items = n_tiles * splits;
        const double t = estimated_us(g);
        if (!found || t < least) *out = g, least = t, found = true;
    }
    out->per_xcd = (out->n_items + 7) / 8;
    return found;
}

// The product on a tile of whole_patch.hip.  false: some column tile's pixels of all channels do not fit LDS.
// *us: its estimated time, a fixed part and per round of workgroups another, the steps of a wavefront, the patch to clear and
// the loader's batches.  Fitted to 1 100 measurements (12 layers of 32 to 384 channels, planes of 8 x 8 to 31 x 31, windows of
// 1, 3 and 5, 1 to 100 images, both directions; mean deviation 3 to 4 %, largest 19 %).  Used beyond those ranges: of 30 000 random
// forward passes (32 to 1 024 channels, 8 to 1 024 filters, planes of 5 x 5 to 64 x 64, windows up to 7, 1 to 64 images) it is 10 %
// low on average, as the larger tiles' estimate is 7 %, and off by a quarter on one in a hundred.  What is chosen takes 0.78 of the
// larger tiles' time there and 1.0075 of the best tile's; 99 passes are more than 3 % slower than on the larger tiles, the
// slowest 22 %.  Two workgroups of the 32 x 64 tile share a compute unit where their LDS allows it; the others' registers or
// wavefronts fill it.
static bool plan_whole_patch(const Geom &base, int config, double limit, Geom *out, double *us)
{
    Geom g = base;
    const WholeTile t = whole_tile(config);
    g.config = config, g.bm = t.bm, g.bn = t.bn;
    g.tiles_f = (g.F + t.bm - 1) / t.bm, g.tiles_m = (g.M + t.bn - 1) / t.bn;  // Fp, the packed weights' order, stays
    if (g.tiles_f * t.bm > g.Fp) return false;  // weights packed for the 96-row tile
    g.splits = 1, g.chunks_per_split = g.n_chunks;
    g.n_items = g.tiles_f * g.tiles_m;
    g.per_xcd = (g.n_items + 7) / 8;
    static const struct { int tasks; double fixed, round, step, clear, batch; } cost[WHOLE_CONFIGS] = {
        {1024, 1.81, 1.78, 0.138, 0.446, 1.78}, {512, 2.73, 1.22, 0.127, 0.32, 0.31},
        {1024, 1.75, 1.85, 0.214, 0.367, 1.85}, {1024, 1.59, 4.49, 0.297, 0.413, 0.384}};
    const auto &c = cost[config];
    const double steps = (g.n_chunks * g.KK + t.waves - 1) / t.waves;
    if (c.fixed + (g.n_items + 511) / 512 * (c.round + c.step * steps) > limit) return false;  // before every tile's pixels are looked at
    g.Wp = g.W + 2 * g.pw;
    // on planes and rows of an even number of elements every 8 of them start at a multiple of 4 bytes
    g.piece = g.HW % 2 == 0 && g.W % 2 == 0 ? 8 : 7;
    const int64_t packs = NG * (int64_t)g.n_chunks, most = WHOLE_LDS / 16 / packs - 1;  // patch pixels per channel pack
    const TileExtent e = tile_extent(g, t.bn, most / g.Wp, 0x7fffffff);
    if (!e.fits) return false;
    const int pieces = g.piece == 8 ? e.pieces8 : e.pieces7;
    g.plane = e.rows * g.Wp | 1;
    // tiles that an XCD's cache serves: those of one row panel, or those of one column tile, whichever operand is larger
    g.cols_fastest = (double)g.Fp * g.C * g.KK > (double)g.N * g.C * g.HW ? 1 : 0;
    g.div_tiles = FastDiv((uint32_t)(g.cols_fastest ? g.tiles_m : g.tiles_f));
    const size_t patch = (size_t)packs * g.plane * 16;
    const bool pairs = config == 1 && (patch > t.lds ? patch : t.lds) <= 80 * 1024, crowded = pairs && g.n_items > 256;
    const int64_t rounds = (g.n_items + (pairs ? 511 : 255)) / (pairs ? 512 : 256);
    const double batches = (double)((packs * pieces + c.tasks - 1) / c.tasks);
    *us = c.fixed + rounds * (c.round + c.step * steps + c.clear * packs * g.plane / (64.0 * t.waves) + c.batch * batches +
                              (crowded ? 1.42 + 0.095 * steps : 0.0));
    *out = g;
    return true;
}

// The plan is a function of the extents and the tuning overrides alone, but checking every tile position of a large
// layer takes 17 us of host time, and a call needs the plan up to three times.  Each thread keeps its last plans by value.
// `masked`: a result in the rows form behind a ReLU's mask, which the tiles of whole_patch.hip do not store: where those pay, the
// larger tiles' reduction is split, and the mask is refused.
static bool make_fused_geom(const ConvGeom &c, bool data_gradient, Geom *g, bool masked = false)
{
    struct Key { int32_t v[16]; };
    struct Entry { Key key; bool used, ok; Geom geom; };
    constexpr int ENTRIES = 64;
    static thread_local Entry cache[ENTRIES];
    const Key key{{c.N, c.C, c.H, c.W, c.F, c.kh, c.kw, c.sh, c.sw, c.ph, c.pw, (data_gradient ? 1 : 0) + (masked ? 2 : 0), g_fused_bn, g_fused_bm, g_fused_bare_pitch, g_fused_whole}};
    uint32_t hash = 0;
    for (int32_t v : key.v) hash = hash * 0x9e3779b1u + (uint32_t)v + (hash >> 15);
    Entry &e = cache[hash % ENTRIES];
    if (!e.used || memcmp(&e.key, &key, sizeof key) != 0) {
        e.key = key, e.used = true;
        e.ok = plan_fused_geom(c, data_gradient, &e.geom);
        e.geom.whole = e.geom.splits == 1 ? 1 : 0;
        const bool few = e.ok && e.geom.tiles_f * e.geom.tiles_m <= 128;  // of the larger tiles
        // the small tile where it is estimated at least 5 % faster (what the estimate is good for); a tuning override of
        // another tile keeps it out, its own override puts it in wherever it fits
        if (e.ok && g_fused_bm == 0 && (g_fused_bn == 0 || g_fused_bn == BN_SMALL)) {
            const double factor = g_fused_bn == BN_SMALL ? 0.0 : 1.05, base = estimated_us(e.geom);
            Geom small;
            if (plan_small_tile(e.geom, &small) && factor * estimated_us(small) < base) e.geom = small;
        }
        // The tiles of whole_patch.hip where estimated at least 10 % faster, for products of few of the larger tiles (beyond them each of its
        // workgroups' own latency weighs more than an even spread: 256 -> 384, 13 x 13, 50 images 32 us on the larger tiles, 35
        // on the best of these); its override keeps them out (1) or puts one in wherever it fits.
        if (e.ok && !masked && g_fused_bn == 0 && g_fused_bm == 0 && (g_fused_whole > 1 || (g_fused_whole == 0 && few))) {
            double best = estimated_us(e.geom) / 1.1, us;
            const Geom base = e.geom;
            Geom whole;
            for (int config = 0; config < WHOLE_CONFIGS; ++config)
                if ((g_fused_whole == 0 || g_fused_whole == config + 2) && plan_whole_patch(base, config, g_fused_whole != 0 ? 1e30 : best, &whole, &us) &&
                    (us < best || g_fused_whole != 0))
                    e.geom = whole, best = us;
        }
    }
    *g = e.geom;
    return e.ok;
}

}  // namespace fused

void set_fused_tile_override(int bn, int bm)
{
    if (bn >= 0) fused::g_fused_bn = bn;
    if (bm >= 0) fused::g_fused_bm = bm;
}
void set_fused_whole_override(int value) { fused::g_fused_whole = value; }
void set_fused_pitch_override(int bare) { fused::g_fused_bare_pitch = bare; }

bool fused_supported(const ConvGeom &c, int dtype, bool data_gradient)
{
    fused::Geom g;
    return dtype == OMNI_BF16 && fused::make_fused_geom(c, data_gradient, &g);
}

static size_t fused_packed_bytes(const fused::Geom &g)
{
    return ((size_t)g.n_chunks * g.KK * fused::NG * g.Fp * 16 + 255) / 256 * 256;
}

// the repacked weights, then (split reductions only) the fp32 partial results [splits][F][M]
size_t fused_weight_bytes(const ConvGeom &c, bool data_gradient)
{
    fused::Geom g;
    if (!fused::make_fused_geom(c, data_gradient, &g)) return 0;
    return fused_packed_bytes(g) + (g.splits > 1 ? (size_t)g.splits * g.F * g.M * sizeof(float) : 0);
}

// The most fused_weight_bytes() can be at any batch up to this one (the other extents the same).  Tiles and splits change
// with the batch, and with them the need goes up and down.  Packed weights: rows rounded up to 128 (96-row tiles take
// fewer).  Sums: at most a copy of the result per chunk, of a result of at most 128 of the widest tiles (a larger one is
// not split), and at most one workgroup per compute unit of 128 x 512 results.
size_t fused_weight_bound(const ConvGeom &c, int dtype, bool data_gradient)
{
    using namespace fused;
    const int C = data_gradient ? c.F : c.C, F = data_gradient ? c.C : c.F;
    if (dtype != OMNI_BF16 || c.sh != 1 || c.sw != 1 || C % CH != 0) return 0;
    if (data_gradient ? (c.kh - 1 < c.ph || c.kw - 1 < c.pw || c.HoWo < 8) : (int64_t)c.H * c.W < 8) return 0;
    const int64_t n_chunks = C / CH, Fp = round_up(F, 128), M = (int64_t)c.N * (data_gradient ? (int64_t)c.H * c.W : c.HoWo);
    const int64_t M_split = 128 / (Fp / 128) * BN_WIDE;
    const double packed = (double)n_chunks * c.kh * c.kw * NG * (double)Fp * 16.0;
    const double copies = n_chunks < 2 ? 0.0 : (double)n_chunks * F * (double)(M < M_split ? M : M_split) * 4.0, chip = 256.0 * 128.0 * BN_WIDE * 4.0;
    return (size_t)(packed + 256.0 + (copies < chip ? copies : chip));
}

static void fill_fused_job(const fused::Geom &g, bool data_gradient, const void *W, void *packed, PackJob *job)
{
    job->kind = 0;
    job->W = (const bf16_t *)W, job->Wt = (uint4 *)packed;
    job->total = (int64_t)g.n_chunks * g.KK * fused::NG * g.Fp;
    job->F = g.F, job->Fp = g.Fp, job->KK = g.KK, job->n_chunks = g.n_chunks, job->flip = data_gradient ? 1 : 0;
    job->stride_out = data_gradient ? g.KK : (int64_t)g.C * g.KK;
    job->stride_in = data_gradient ? (int64_t)g.F * g.KK : g.KK;
    job->C = job->kh = job->kw = job->kwq = job->groups = job->BM = 0;
}

bool fused_pack_job(const ConvGeom &c, bool data_gradient, const void *W, void *packed, PackJob *job, size_t *bytes)
{
    fused::Geom g;
    *bytes = 0;
    if (!fused::make_fused_geom(c, data_gradient, &g)) return false;
    *bytes = fused_packed_bytes(g);
    if (job != nullptr) fill_fused_job(g, data_gradient, W, packed, job);
    return true;
}

int launch_pack_jobs(const PackJobTable &t, hipStream_t s)
{
    if (t.n <= 0) return OMNI_OK;
    double bytes = 0.0;
    for (int j = 0; j < t.n; ++j) bytes += 2.0 * 16.0 * (double)t.job[j].total;
    ProfScope prof(KID_PACK_KHAT, s, 0.0, bytes);
    hipLaunchKernelGGL(fused::pack_jobs_kernel, dim3((unsigned)t.first_block[t.n]), dim3(256), 0, s, t);
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
}

int fused_column_tiles(const ConvGeom &c, bool data_gradient)
{
    fused::Geom g;
    if (!fused::make_fused_geom(c, data_gradient, &g, true) || !g.whole) return 0;
    return g.tiles_m;
}

// `prepacked` != null: the repacked weights already exist there (fused_pack_job) and W is not read.
// io (optional): in_ld > 0 = the input is not the dense tensor but its rows form, a matrix [C][in_ld] with image n's
// plane of channel c at column n * (the plane rounded up to 8 elements); mask != null = the output is written in
// the rows form too (leading dimension out_ld), zero where the dense tensor `mask` [N][F][Ho][Wo] is not positive,
// with col_sums [F][fused_column_tiles] (nullable) receiving every column tile's sums of the stored values.
int launch_fused_conv(const ConvGeom &c, bool data_gradient, const void *X, const void *W, const float *bias,
                      int relu, void *Y, void *wt_scratch, hipStream_t s, int kid, const void *prepacked, const FusedIO *io)
{
    using namespace fused;
    const int64_t in_ld = io != nullptr ? io->in_ld : 0;
    const bool masked = io != nullptr && io->mask != nullptr;
    Geom g;
    if (!make_fused_geom(c, data_gradient, &g, masked)) return OMNI_UNSUPPORTED;
    const int64_t out_pitch = ((int64_t)g.HoWo + 7) / 8 * 8;
    if (masked && (in_ld <= 0 || !g.whole || bias != nullptr || relu || io->out_ld < g.N * out_pitch ||
                   (double)io->out_ld * g.F * 2.0 >= 4.0e9))
        return OMNI_UNSUPPORTED;
    if (in_ld > 0) {
        const int64_t pitch = ((int64_t)g.HW + 7) / 8 * 8;
        if (in_ld < g.N * pitch || in_ld % 2 != 0 || (double)in_ld * g.C * 2.0 >= 4.0e9) return OMNI_UNSUPPORTED;  // (it is a multiple of 64)
        g.sn = (uint32_t)pitch, g.sc = (uint32_t)in_ld;
    }
    if (prepacked == nullptr) {
        PackJobTable t;
        fill_fused_job(g, data_gradient, W, wt_scratch, &t.job[0]);
        t.first_block[0] = 0, t.first_block[1] = (t.job[0].total + 255) / 256, t.n = 1;
        int st = launch_pack_jobs(t, s);
        if (st != OMNI_OK) return st;
    }
    const bf16_t *wt = (const bf16_t *)(prepacked != nullptr ? prepacked : wt_scratch);
    FwdEpilogue<bf16_t> epi{(bf16_t *)Y, bias, g.F, g.M, g.HoWo, g.div_HoWo, relu};
    ProfScope prof(kid >= 0 ? kid : (data_gradient ? KID_FUSED_DGRAD : KID_FUSED_FWD), s, 2.0 * (double)c.M * c.K * c.F, 0.0);
    dim3 grid((unsigned)(g.per_xcd * 8)), block(g.bm == 64 ? 256 : 512);
    float *partials = reinterpret_cast<float *>(reinterpret_cast<char *>(wt_scratch) + fused_packed_bytes(g));
    PartialEpilogue pe{partials, g.F, g.M};
    RowsMaskEpilogue me{(bf16_t *)Y, masked ? (const bf16_t *)io->mask : nullptr, masked ? io->col_sums : nullptr, g.F, g.M, g.HoWo,
                        g.div_HoWo, (uint32_t)out_pitch, masked ? (uint32_t)io->out_ld : 0u};
#define OMNI_FUSED_LAUNCH_IN(BM_, WM_, WN_, BN_, PATCH_, RIN_, SWZ_)                                                         \
    do {                                                                                                                    \
        if (g.splits > 1)                                                                                                   \
            hipLaunchKernelGGL((fused_conv_kernel<BM_, WM_, WN_, BN_, PATCH_, PartialEpilogue, RIN_, SWZ_>), grid, block, 0, \
                               s, (const bf16_t *)X, wt, g, pe);                                                            \
        else                                                                                                                \
            hipLaunchKernelGGL((fused_conv_kernel<BM_, WM_, WN_, BN_, PATCH_, FwdEpilogue<bf16_t>, RIN_, SWZ_>), grid,      \
                               block, 0, s, (const bf16_t *)X, wt, g, epi);                                                 \
    } while (0)
#define OMNI_FUSED_LAUNCH(BM_, WM_, WN_, BN_, PATCH_)                                                                       \
    do {                                                                                                                    \
        if (masked)                                                                                                         \
            hipLaunchKernelGGL((fused_conv_kernel<BM_, WM_, WN_, BN_, PATCH_, RowsMaskEpilogue, true>), grid, block, 0, s,   \
                               (const bf16_t *)X, wt, g, me);                                                               \
        else if (in_ld > 0) OMNI_FUSED_LAUNCH_IN(BM_, WM_, WN_, BN_, PATCH_, true, false);                                  \
        else if (g.piece == 8) OMNI_FUSED_LAUNCH_IN(BM_, WM_, WN_, BN_, PATCH_, false, true);                               \
        else OMNI_FUSED_LAUNCH_IN(BM_, WM_, WN_, BN_, PATCH_, false, false);                                                \
    } while (0)
    if (g.config >= 0) launch_whole_patch(g, in_ld > 0, (const bf16_t *)X, wt, epi, s);
    else if (g.bm == 64) OMNI_FUSED_LAUNCH(64, 2, 2, BN_SMALL, PATCH_SMALL);
    else if (g.bm == 96) OMNI_FUSED_LAUNCH(96, 1, 8, BN_WIDE, PATCH_WIDE);
    else if (g.bn == BN_WIDE) OMNI_FUSED_LAUNCH(128, 2, 4, BN_WIDE, PATCH_WIDE);
    else if (g.bn == BN_MID) OMNI_FUSED_LAUNCH(128, 2, 4, BN_MID, PATCH_MID);
    else OMNI_FUSED_LAUNCH(128, 2, 4, BN_NARROW, PATCH_NARROW);
#undef OMNI_FUSED_LAUNCH
#undef OMNI_FUSED_LAUNCH_IN
    OMNI_LAUNCH_CHECK();
    if (g.splits > 1) launch_reduce_store(partials, g.splits, g.F, g.M, epi, s);
    OMNI_LAUNCH_CHECK();
    return OMNI_OK;
}

}  // namespace omni

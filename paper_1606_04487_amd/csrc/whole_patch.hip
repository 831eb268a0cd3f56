// Fused convolution for products of few tiles (gfx950, bf16, stride 1): the same product as implicit.hip's
// fused_conv_kernel, laid out for latency instead of throughput.
//
// With few images a layer has fewer of the large tiles than the chip has compute units.  Cutting the reduction over
// several workgroups per tile fills the chip, but costs fp32 sums in memory and a launch that adds them, and each
// workgroup still walks its channels one chunk at a time: pixels, barrier, weights, barrier.  Here a workgroup takes a
// small tile and ALL channels: it brings the pixels its columns touch of every channel into LDS at once (one memory
// latency, one barrier), then its wavefronts divide the reduction steps (chunk, tap) among themselves.  Each of them
// holds the whole tile's sums and reads the weights of its steps straight from memory into registers, several steps
// ahead: no two wavefronts share a step, so staging them in LDS would save nothing, and there is no barrier until all
// steps are done.  The wavefronts' sums are then added through LDS in a fixed order, and each 32 x 32 piece of the
// result is stored by one of them through the common staged epilogue.
//
// Bound by latencies, a chain of them: kernel arguments and tile geometry 1.3 us, pixels 1.2, steps 0.1 to 0.3 each, sums
// 1, store 0.6 (one workgroup per compute unit).  Measured, product and sum of a split one together: 256 -> 384 channels,
// 13 x 13, window 3, one image 9.9 -> 7.2 us, four 13.1 -> 8.5, sixteen 22.4 -> 15.0; 96 -> 256, 27 x 27, window 5, one image
// 12.4 -> 7.7; 32 -> 32, 16 x 16, window 5, fifty 9.7 -> 5.2; 635 random layers and directions 0.80 of the time on average.
//
// Layout of the patch: [8-channel pack][pixel] of 16-byte packs as in fused_conv_kernel, pixels in plain order.  The
// planes are an odd number of packs apart, so that the transposing stores, whose neighbouring lanes hold neighbouring
// channel packs, fall on different banks.
//
// A 16-byte load from an address that is only 2-byte aligned costs a wavefront 65 cycles, from a multiple of 4 bytes 20,
// and on odd planes half of the channels' rows are of the slow kind.  So a loader task takes 7 elements there: each
// channel's 8 start at the 4-byte boundary at or before them and are shifted by one element where they have to be.  The
// element that such a load reads beyond its plane's end belongs to the next plane; the tensor ends on a 4-byte boundary
// (its channels are a multiple of 32), where the load starts early, so nothing beyond it is read.
#include "common.h"
#include "fused_geom.h"
#include "mma_epilogue.h"

namespace omni {
namespace fused {

// Adding the wavefronts' sums: [wavefront][row][column] with rows of BN + 4 fp32, an odd number of 16-byte packs.  Where
// that is more than LDS holds, the upper half of the wavefronts adds its sums to the lower half's first.
constexpr int whole_pitch(int TJ) { return 32 * TJ + 4; }
constexpr int whole_folds(int TI, int TJ, int NW) { return NW * 32 * TI * whole_pitch(TJ) * 4 > (int)WHOLE_LDS ? 1 : 0; }
constexpr int whole_lds_bytes(int TI, int TJ, int NW) { return (NW >> whole_folds(TI, TJ, NW)) * 32 * TI * whole_pitch(TJ) * 4; }

// The lower (upper) halves of a and b as one word.
__device__ __forceinline__ uint32_t pick_lo(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); }
__device__ __forceinline__ uint32_t pick_hi(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

// V neighbouring results x of row i from column j on, through the epilogue to memory.
template <int V>
__device__ __forceinline__ void store_piece(const FwdEpilogue<bf16_t> &epi, int i, int j, const float (&x)[V], float add)
{
    if (i >= epi.n_rows()) return;
    bool ok0, ok1;
    const uint32_t rs = epi.row_stride32(), off0 = epi.col_off32(j, ok0), off1 = epi.col_off32(j + V - 1, ok1);
    char *row = epi.base32(0) + (int64_t)i * rs;
    float y[V];
#pragma unroll
    for (int e = 0; e < V; ++e) y[e] = epi.apply(x[e], add);
    if (ok0 && ok1 && off1 - off0 == (uint32_t)((V - 1) * 2)) {
        uint32_t w[V / 2];
#pragma unroll
        for (int e = 0; e < V; e += 2) w[e / 2] = f32x2_to_bf16x2(y[e], y[e + 1]);
        __builtin_memcpy(row + off0, w, sizeof w);  // element-aligned
    } else {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            bool ok;
            const uint32_t off = epi.col_off32(j + e, ok);
            if (ok) *reinterpret_cast<bf16_t *>(row + off) = f32_to_bf16(y[e]);
        }
    }
}

// TI x TJ: 32 x 32 pieces of the tile; NW: wavefronts; D: steps whose weights are in flight (even); B: loader tasks whose
// pixels are in flight per thread; WPE: wavefronts per SIMD that the register budget leaves room for.
template <int TI, int TJ, int NW, int D, int B, int WPE, bool RIN>
__global__ __launch_bounds__(64 * NW, WPE) void whole_patch_kernel(const bf16_t *__restrict__ X, const bf16_t *__restrict__ Wt,
                                                                   Geom g, FwdEpilogue<bf16_t> epi)
{
    constexpr int NT = 64 * NW, BM = 32 * TI, BN = 32 * TJ;
    static_assert(D % 2 == 0, "two sets of pixel fragments take turns");
    extern __shared__ __align__(16) uint4 whole_smem[];

    const int item = (blockIdx.x % 8) * g.per_xcd + blockIdx.x / 8;  // contiguous ranges of tiles per XCD
    if (item >= g.n_items) return;
    int tm, tf;
    if (g.cols_fastest) tf = (int)g.div_tiles.div((uint32_t)item), tm = item - tf * g.tiles_m;
    else tm = (int)g.div_tiles.div((uint32_t)item), tf = item - tm * g.tiles_f;
    const int row0 = tf * BM, col0 = tm * BN;
    const int m_last = (col0 + BN < g.M ? col0 + BN : g.M) - 1;
    const int n0 = (int)g.div_HoWo.div((uint32_t)col0);
    const int nslots = (int)g.div_HoWo.div((uint32_t)m_last) - n0 + 1;
    const int tid = threadIdx.x, lane = tid % 64, wave = __builtin_amdgcn_readfirstlane(tid / 64);
    const int li = lane % 32, h = lane / 32;

    // The images the columns lie in, one after the other: padded rows from patch row `so` on, loader pieces from p0 on.
    const int piece = g.piece;
    auto n_pieces = [&](int len) { return piece == 8 ? (len + 7) >> 3 : (int)__umulhi((uint32_t)(len + 6), 613566757u); };
    int PT = 0;
    for (int i = 0; i < nslots; ++i) PT += n_pieces(slot_span(g, col0, m_last, n0 + i).len);

    // A loader task is 8 channels (one pack) x `piece` consecutive elements of one image's rows: eight 16-byte loads,
    // transposed in registers to one pack per pixel.  Neighbouring lanes take the four packs of a chunk, then the next piece.
    const int packs = NG * g.n_chunks, tasks = packs * PT;
    const float inv_PT = __builtin_amdgcn_rcpf((float)(PT > 0 ? PT : 1));
    const uint32_t plane_e = RIN ? g.sc : (uint32_t)g.HW;
    const char *xb = reinterpret_cast<const char *>(X);
    u32x4 *const patch = reinterpret_cast<u32x4 *>(whole_smem);
    u32x4 r[B][8];
    int dst[B], x0[B], lo[B], hi[B];  // LDS pack of element 0, its column, and which elements the task has
    uint32_t odd[B];                  // bit e: channel e's load starts one element early
    auto issue = [&](auto b, int t) {
        constexpr int I = decltype(b)::value;
        lo[I] = hi[I] = 0, dst[I] = 0, x0[I] = 0, odd[I] = 0;
        if (t - lane >= tasks) return;  // nothing for any lane of the wavefront
        if (t >= tasks) return;
        const int rest = t / NG, quad = (int)(((float)rest + 0.5f) * inv_PT), jj = rest - quad * PT, pk = quad * NG + t % NG;
        int so = 0, p0 = 0, my_n = 0, my_so = 0, my_j = 0, my_ya = 0, my_len = 0, my_ra = 0;
        for (int i = 0; i < nslots; ++i) {
            const SlotSpan s = slot_span(g, col0, m_last, n0 + i);
            if (jj >= p0) my_n = n0 + i, my_so = so, my_j = jj - p0, my_ya = s.ya, my_len = s.len, my_ra = s.ra;
            so += s.nrows, p0 += n_pieces(s.len);
        }
        const int ea = my_ya * g.W, eb = ea + my_len;
        int e0 = ea + piece * my_j;
        e0 = e0 < g.HW - piece ? e0 : g.HW - piece;  // stay inside the plane: the overlap rewrites equal values
        uint32_t y, x;
        g.div_W.divmod((uint32_t)e0, y, x);
        dst[I] = pk * g.plane + (my_so + (int)y + g.ph - my_ra) * g.Wp + (int)x + g.pw;
        x0[I] = (int)x, lo[I] = ea - e0, hi[I] = eb - e0 < piece ? eb - e0 : piece;
        uint32_t at;  // element of channel 0's load
        if constexpr (RIN) at = (uint32_t)my_n * g.sn + (uint32_t)(8 * pk) * g.sc + (uint32_t)e0;
        else at = (uint32_t)(my_n * g.C + 8 * pk) * (uint32_t)g.HW + (uint32_t)e0;
        odd[I] = at & 1u;  // of channel 0; channel e's is this plus e times the plane's
#pragma unroll
        for (int e = 0; e < 8; ++e, at += plane_e) __builtin_memcpy(&r[I][e], __builtin_assume_aligned(xb + (at & ~1u) * 2u, 4), 16);
    };
    auto commit = [&](auto b) {
        constexpr int I = decltype(b)::value;
        if (__builtin_amdgcn_ballot_w64(hi[I] > lo[I]) == 0) return;
        if (piece != 8) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint32_t sh = ((odd[I] + (uint32_t)e * plane_e) & 1u) * 16u;
#pragma unroll
                for (int w = 0; w < 3; ++w) r[I][e][w] = __builtin_amdgcn_alignbit(r[I][e][w + 1], r[I][e][w], sh);
                r[I][e][3] >>= sh;
            }
        }
        int d = dst[I], x = x0[I];
        static_for<0, 8>([&](auto ee) {
            constexpr int e = decltype(ee)::value, w = e / 2;
            u32x4 v;
            if constexpr (e % 2 == 0)
                v = u32x4{pick_lo(r[I][0][w], r[I][1][w]), pick_lo(r[I][2][w], r[I][3][w]), pick_lo(r[I][4][w], r[I][5][w]), pick_lo(r[I][6][w], r[I][7][w])};
            else
                v = u32x4{pick_hi(r[I][0][w], r[I][1][w]), pick_hi(r[I][2][w], r[I][3][w]), pick_hi(r[I][4][w], r[I][5][w]), pick_hi(r[I][6][w], r[I][7][w])};
            if (e >= lo[I] && e < hi[I]) patch[d] = v;
            ++d;
            if (++x == g.W) x = 0, d += g.Wp - g.W;
        });
    };
    static_for<0, B>([&](auto b) { issue(b, tid + decltype(b)::value * NT); });

    // This wavefront's steps (chunk, tap) and the weights of the first D of them.  A step's weight tile is [g][Fp] packs.
    const int KK = g.KK, n_steps = g.n_chunks * KK;
    const int st_lo = wave * n_steps / NW, st_hi = (wave + 1) * n_steps / NW;
    const char *const wt = reinterpret_cast<const char *>(Wt);
    const uint32_t wt_lane = (uint32_t)(h * g.Fp + row0 + li) * 16u, half_b = (uint32_t)g.Fp * 32u;
    const int64_t step_b = (int64_t)g.Fp * (NG * 16);
    uint4 fa[D][2][TI];
    auto issue_a = [&](auto q, int st) {
        constexpr int Q = decltype(q)::value;
        st = st < st_hi ? st : st_hi - 1;   // beyond the last one: repeats it, unused
        st = st < 0 ? 0 : st;
        const char *p = wt + st * step_b;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int t = 0; t < TI; ++t) fa[Q][s2][t] = *reinterpret_cast<const uint4 *>(p + (wt_lane + s2 * half_b) + t * 512);
    };
    static_for<0, D>([&](auto q) { issue_a(q, st_lo + decltype(q)::value); });

    // everything outside the real pixels stays zero: loads only ever write real pixels
    for (int i = tid; i < packs * g.plane; i += NT) whole_smem[i] = make_uint4(0, 0, 0, 0);

    // patch pixel of each of this lane's columns at tap (0, 0)
    int pb[TJ];
#pragma unroll
    for (int u = 0; u < TJ; ++u) {
        int m = col0 + 32 * u + li;
        m = m < g.M ? m : g.M - 1;
        uint32_t n, q, oy, ox;
        g.div_HoWo.divmod((uint32_t)m, n, q);
        g.div_Wo.divmod(q, oy, ox);
        int so = 0, my_so = 0, my_ra = 0;
        for (int i = 0; i < nslots; ++i) {
            const SlotSpan s = slot_span(g, col0, m_last, n0 + i);
            if ((int)n - n0 == i) my_so = so, my_ra = s.ra;
            so += s.nrows;
        }
        pb[u] = (my_so + (int)oy - my_ra) * g.Wp + (int)ox + h * g.plane;
    }
    __syncthreads();
    static_for<0, B>([&](auto b) { commit(b); });
    for (int t = tid + B * NT; t - tid < tasks; t += B * NT) {
        static_for<0, B>([&](auto b) { issue(b, t + decltype(b)::value * NT); });
        static_for<0, B>([&](auto b) { commit(b); });
    }
    __syncthreads();

    // The products are transposed: a lane's registers hold neighbouring columns of one row, which is how the sums are
    // added and stored.
    f32x16 acc[TI][TJ];
#pragma unroll
    for (int t = 0; t < TI; ++t)
#pragma unroll
        for (int u = 0; u < TJ; ++u)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][u][v] = 0.f;

    int chunk = st_lo / KK, ky = (st_lo - chunk * KK) / g.kw, kx = st_lo - chunk * KK - ky * g.kw;
    int off = chunk * NG * g.plane + ky * g.Wp + kx;
    const int half_p = 2 * g.plane;
    auto advance = [&]() {
        ++off;
        if (++kx == g.kw) {
            kx = 0, off += g.Wp - g.kw;
            if (++ky == g.kh) ky = 0, ++chunk, off = chunk * NG * g.plane;
        }
    };
    uint4 fb[2][2][TJ];
    auto load_b = [&](auto q) {
        constexpr int Q = decltype(q)::value;
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int u = 0; u < TJ; ++u) fb[Q][s2][u] = whole_smem[pb[u] + off + s2 * half_p];
    };
    auto step = [&](auto q, int st, bool more) {
        constexpr int Q = decltype(q)::value;
        if (more) {
            advance();
            load_b(std::integral_constant<int, (Q + 1) & 1>{});
            __builtin_amdgcn_sched_barrier(0);  // the next step's fragments are read under this step's products
        }
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
            for (int t = 0; t < TI; ++t)
#pragma unroll
                for (int u = 0; u < TJ; ++u) Mma<bf16_t>::run(fb[Q & 1][s2][u], fa[Q][s2][t], acc[t][u]);
        issue_a(q, st + D);
    };
    if (st_lo < st_hi) load_b(std::integral_constant<int, 0>{});
    int st = st_lo;
    for (; st + D < st_hi; st += D) static_for<0, D>([&](auto q) { step(q, st + decltype(q)::value, true); });
    static_for<0, D>([&](auto q) {
        if (st + decltype(q)::value < st_hi) step(q, st + decltype(q)::value, st + decltype(q)::value + 1 < st_hi);
    });

    // The wavefronts' sums, added in the order of the wavefronts.
    constexpr int FOLD = whole_folds(TI, TJ, NW), H = NW >> FOLD, PITCH = whole_pitch(TJ);
    typedef float f32x4 __attribute__((ext_vector_type(4)));
    float *const sums = reinterpret_cast<float *>(whole_smem);
    auto quad = [&](int w, int t, int u, int v) {  // result columns 32u + 8v + 4h .. + 3 of row 32t + li
        return reinterpret_cast<f32x4 *>(sums + (w * BM + 32 * t + li) * PITCH + 32 * u + 8 * v + 4 * h);
    };
    auto put = [&](int w) {
#pragma unroll
        for (int t = 0; t < TI; ++t)
#pragma unroll
            for (int u = 0; u < TJ; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    *quad(w, t, u, v) = f32x4{acc[t][u][4 * v], acc[t][u][4 * v + 1], acc[t][u][4 * v + 2], acc[t][u][4 * v + 3]};
    };
    // a thread's pieces of V results of one row, and the row terms that belong to them
    constexpr int V = BM * BN / 8 < NT ? 4 : 8, GPR = BN / V, PIECES = BM * GPR, PER = (PIECES + NT - 1) / NT;
    static_assert(V == 4 || V == 8, "8 or 16 bytes of bf16");
    float add[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int q = tid + p * NT;
        add[p] = PIECES % NT == 0 || q < PIECES ? epi.row_add(row0 + q / GPR) : 0.f;
    }
    __syncthreads();  // every wavefront has read its last pixels
    if constexpr (FOLD) {
        if (wave >= H) put(wave - H);
        __syncthreads();
        if (wave < H) {
#pragma unroll
            for (int t = 0; t < TI; ++t)
#pragma unroll
                for (int u = 0; u < TJ; ++u)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const f32x4 f = *quad(wave, t, u, v);
                        const f32x4 s = {acc[t][u][4 * v] + f[0], acc[t][u][4 * v + 1] + f[1], acc[t][u][4 * v + 2] + f[2], acc[t][u][4 * v + 3] + f[3]};
                        *quad(wave, t, u, v) = s;  // the place it has just read
                    }
        }
    } else {
        put(wave);
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int q = tid + p * NT, i = q / GPR, j = q % GPR * V;
        if (PIECES % NT != 0 && q >= PIECES) continue;
        float x[V];
#pragma unroll
        for (int e = 0; e < V; e += 4) {
            f32x4 f[H];
#pragma unroll
            for (int w = 0; w < H; ++w) f[w] = *reinterpret_cast<const f32x4 *>(sums + (w * BM + i) * PITCH + j + e);
#pragma unroll
            for (int w = 1; w < H; ++w) f[0] += f[w];
            x[e] = f[0][0], x[e + 1] = f[0][1], x[e + 2] = f[0][2], x[e + 3] = f[0][3];
        }
        store_piece<V>(epi, row0 + i, col0 + j, x, add[p]);
    }
}

WholeTile whole_tile(int config)
{
    switch (config) {
    case 0: return {32, 32, 16, whole_lds_bytes(1, 1, 16)};
    case 1: return {32, 64, 8, whole_lds_bytes(1, 2, 8)};
    case 2: return {64, 64, 8, whole_lds_bytes(2, 2, 8)};
    default: return {64, 96, 8, whole_lds_bytes(2, 3, 8)};
    }
}

template <int TI, int TJ, int NW, int D, int B, int WPE>
static void launch_config(const Geom &g, bool rows_in, const bf16_t *X, const bf16_t *wt, const FwdEpilogue<bf16_t> &epi, hipStream_t s)
{
    const size_t patch = (size_t)NG * g.n_chunks * g.plane * 16, sums = whole_lds_bytes(TI, TJ, NW);
    const unsigned lds = (unsigned)(patch > sums ? patch : sums);
    const dim3 grid((unsigned)(g.per_xcd * 8)), block(64 * NW);
    if (rows_in) hipLaunchKernelGGL((whole_patch_kernel<TI, TJ, NW, D, B, WPE, true>), grid, block, lds, s, X, wt, g, epi);
    else hipLaunchKernelGGL((whole_patch_kernel<TI, TJ, NW, D, B, WPE, false>), grid, block, lds, s, X, wt, g, epi);
}

void launch_whole_patch(const Geom &g, bool rows_in, const bf16_t *X, const bf16_t *wt, const FwdEpilogue<bf16_t> &epi, hipStream_t s)
{
    switch (g.config) {
    case 0: return launch_config<1, 1, 16, 6, 1, 4>(g, rows_in, X, wt, epi, s);
    case 1: return launch_config<1, 2, 8, 4, 1, 4>(g, rows_in, X, wt, epi, s);
    case 2: return launch_config<2, 2, 8, 4, 2, 2>(g, rows_in, X, wt, epi, s);
    default: return launch_config<2, 3, 8, 4, 2, 2>(g, rows_in, X, wt, epi, s);
    }
}

}  // namespace fused
}  // namespace omni

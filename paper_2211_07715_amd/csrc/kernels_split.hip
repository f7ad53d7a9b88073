// The split-reduction kernel of the sparse INT8 linear layer (gfx950): for
// few tokens (a batch of one sequence), where one workgroup per output tile
// walking the whole reduction would leave most of the chip idle and put
// every window's memory latency in series.
//
// Same product as the other kernels (Section "Sparse GEMM operators", Figure
// 1, Algorithm 1), from the dense operand image (kernels_panel.hip says why;
// here it also halves a wave's load instructions, six of 16 bytes a lane for a
// window instead of ten). A workgroup owns one work item (ST 16-token subtiles
// x NT 16-channel tiles) and splits its reduction over its waves: wave v of kw
// takes windows v, v + kw, ... (at most WPW of them). It issues every load of
// its windows at once -- no lookup stands between a wave and its loads -- and
// so waits about one
// memory latency before its matrix instructions. The waves' int32 partial sums meet in
// LDS; integer addition is exact in any order, so the sum equals the single
// accumulation of the other kernels bit for bit. Each (tile, subtile) pair
// is then reduced, and its epilogue run, by one wave.
//
// What bounds it: a launch's fixed cost (about 2 us back to back) and one
// memory round trip; 4:2-sparse operands -> dense, us at 128 tokens, 80 %: QKV
// 3.47 -> 3.33, attention output 2.76 -> 2.68, FFN1 4.11 -> 3.92, FFN2 3.80 ->
// 3.56.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "sl_device.h"

namespace sl {

// XL: where the rows of x lie; YT: y in SL_LAYOUT_T16X32 (int8 kinds). The
// workgroup has a.kw waves of at most WPW windows each (a.kw * WPW >= n_win).
template <int KIND, int ST, int NT, int WPW, RowsAt XL, bool YT>
__device__ __forceinline__ void split_body(const LinearArgs &a, const GeluArg *ep)
{
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int kw = a.kw;  // = blockDim.x / 64

    // channel-group-major items: the token tiles of one channel group run
    // on one XCD, which then fetches that group's weight operands once
    // (n_items < 2^31)
    const uint32_t item = (uint32_t)xcd_work_index(blockIdx.x, gridDim.x);
    const uint32_t n_mt = (uint32_t)((a.m + 16 * ST - 1) / (16 * ST));
    const int32_t cg = (int32_t)(item / n_mt);
    const int64_t t0 = (int64_t)(item - (uint32_t)cg * n_mt) * (16 * ST);
    const int32_t tile0 = cg * NT;
    const int32_t ntl = min(NT, a.n_tiles - tile0);

    // LDS: the partial sums ([kw][NT*ST] accumulator groups of 64 lanes),
    // then the GELU table
    i32x4 *part = reinterpret_cast<i32x4 *>(smem);
    GeluCell *tab = reinterpret_cast<GeluCell *>(smem + kw * NT * ST * 1024);
    // (rows at whole words change lanes there before this wave's sums go there)
    int8_t *const scratch = smem + wave * NT * ST * 1024;
    // this wave's windows: w_j = wave + j * kw, j < nw
    const int nw = wave < a.n_win ? (a.n_win - 1 - wave) / kw + 1 : 0;

    const __amdgpu_buffer_rsrc_t wr = __builtin_amdgcn_make_buffer_rsrc((void *)a.dense, 0, (int)a.dense_bytes,
                                                                        kRsrcWord3);
    const RowSource<XL> src(a);
    const uint32_t wstride = (uint32_t)a.n_tiles * kDenseOp;  // image bytes per window

    // Token rows: lane l of subtile s loads features 16*(l/16) .. +15 of
    // each half of the window for token (l % 16) -- the B operand layout (tokens past m
    // read zeros or a padding token of the last block, a ragged last window
    // bytes that meet zero weights).
    uint32_t ro[ST];
#pragma unroll
    for (int s = 0; s < ST; ++s) ro[s] = src.offset(a, t0 + s * 16 + src.load_token(lane), src.load_group(lane));

    RowPiece<XL> bv[WPW][ST];
    i32x4 av[WPW][NT][2];
#pragma unroll
    for (int j = 0; j < WPW; ++j) {
        if (j < nw) {
            const uint32_t w = (uint32_t)(wave + j * kw);
#pragma unroll
            for (int s = 0; s < ST; ++s) bv[j][s] = src.load(ro[s], (int)w);
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                // (a tile past the last one reads the last one's: its sums are not used)
                const uint32_t base = (uint32_t)(tile0 + min(c, ntl - 1)) * kDenseOp + 16u * (uint32_t)lane;
#pragma unroll
                for (int h = 0; h < 2; ++h)
                    av[j][c][h] = __builtin_bit_cast(
                        i32x4, __builtin_amdgcn_raw_buffer_load_b128(wr, base + 1024u * h, w * wstride, 0));
            }
        }
    }

    // While those loads are in flight: the epilogue's weight scales and
    // biases of this wave's first (tile, subtile) pair (pair p = (tile c,
    // subtile s) goes to wave p % kw: a workgroup may have fewer waves than
    // pairs), and the GELU step table into LDS.
    auto load_vec = [&](int p, i32x4 &sw, i32x4 &b4) {
        const int32_t ch0 = (tile0 + p / ST) * kTileN + 4 * (lane >> 4);
        const __amdgpu_buffer_rsrc_t sr = __builtin_amdgcn_make_buffer_rsrc((void *)a.w_scale, 0, a.n * 4, kRsrcWord3);
        const __amdgpu_buffer_rsrc_t br = __builtin_amdgcn_make_buffer_rsrc((void *)a.bias, 0, a.n * 4, kRsrcWord3);
        const uint32_t off = ch0 < a.n ? (uint32_t)ch0 * 4u : kOob;
        sw = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(sr, off, 0, 0));
        b4 = __builtin_bit_cast(i32x4, __builtin_amdgcn_raw_buffer_load_b128(br, off, 0, 0));
    };
    i32x4 sw0 = {0, 0, 0, 0}, b40 = {0, 0, 0, 0};
    if constexpr (KIND != SL_EPI_ACC_I32)
        if (wave < NT * ST) load_vec(wave, sw0, b40);
    float hinv = 0.0f, eoff = 0.0f, cmax = 0.0f;
    if constexpr (KIND == SL_EPI_I8_GELU) {
        for (int u = tid; u < ep->nc; u += (int)blockDim.x) tab[u] = ep->cell[u];
        hinv = ep->hinv;
        eoff = ep->off;
        cmax = kGeluBase + (float)(ep->nc - 1);
    }

    i32x4 acc[NT][ST];
#pragma unroll
    for (int c = 0; c < NT; ++c)
#pragma unroll
        for (int s = 0; s < ST; ++s) acc[c][s] = i32x4{0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < WPW; ++j) {
        if (j < nw) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                i32x4 rows[ST];
#pragma unroll
                for (int s = 0; s < ST; ++s) rows[s] = src.operand(bv[j][s], h, ro[s], scratch, lane);
#pragma unroll
                for (int c = 0; c < NT; ++c)
#pragma unroll
                    for (int s = 0; s < ST; ++s)
                        acc[c][s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(av[j][c][h], rows[s], acc[c][s], 0, 0, 0);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < NT; ++c)
#pragma unroll
        for (int s = 0; s < ST; ++s) part[((wave * NT + c) * ST + s) * 64 + lane] = acc[c][s];
    __syncthreads();

    // accumulator layout: lane l holds rows 4*(l/16)+r (channels of one
    // block-row), column l%16 (token), r = 0..3
    for (int p = wave; p < NT * ST; p += kw) {
        const int c = p / ST, s = p % ST;
        if (c < ntl) {
            i32x4 sum = part[(c * ST + s) * 64 + lane];
            for (int v = 1; v < kw; ++v) sum += part[((v * NT + c) * ST + s) * 64 + lane];
            const int32_t ch0 = (tile0 + c) * kTileN + 4 * (lane >> 4);
            const int64_t tok = t0 + s * 16 + (lane & 15);
            float sc[4] = {0.0f, 0.0f, 0.0f, 0.0f}, bb[4] = {0.0f, 0.0f, 0.0f, 0.0f};
            if constexpr (KIND != SL_EPI_ACC_I32) {
                i32x4 sw = sw0, b4 = b40;
                if (p != wave) load_vec(p, sw, b4);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    sc[r] = a.sx * __int_as_float(sw[r]);
                    bb[r] = __int_as_float(b4[r]);
                }
            }
            if (ch0 < a.n) epilogue_store<KIND, YT>(a, sum, tok, ch0, sc, bb, tab, hinv, eoff, cmax);
        }
    }
}

template <int KIND, int ST, int NT, int WPW, RowsAt XL, bool YT>
__global__ __launch_bounds__(64 * kSplitMaxWaves) void sparse_linear_split_kernel(LinearArgs a)
{
    split_body<KIND, ST, NT, WPW, XL, YT>(a, nullptr);
}

template <int ST, int NT, int WPW, RowsAt XL, bool YT>
__global__ __launch_bounds__(64 * kSplitMaxWaves) void sparse_linear_split_gelu_kernel(LinearArgs a, GeluArg ep)
{
    split_body<SL_EPI_I8_GELU, ST, NT, WPW, XL, YT>(a, &ep);
}

template <int KIND, int WPW, RowsAt XL, bool YT>
static sl_status launch_split_wpw(const LinearArgs &a, const GeluArg *ep, hipStream_t stream)
{
    constexpr int ST = kSplitSt, NT = kSplitNt;
    const size_t lds = (size_t)a.kw * NT * ST * 1024 + (KIND == SL_EPI_I8_GELU ? kGeluLds : 0);
    const dim3 grid((uint32_t)a.n_items), block((uint32_t)(64 * a.kw));
    if constexpr (KIND == SL_EPI_I8_GELU)
        hipLaunchKernelGGL((sparse_linear_split_gelu_kernel<ST, NT, WPW, XL, YT>), grid, block, lds, stream, a, *ep);
    else
        hipLaunchKernelGGL((sparse_linear_split_kernel<KIND, ST, NT, WPW, XL, YT>), grid, block, lds, stream, a);
    HIP_TRY(hipGetLastError());
    return SL_OK;
}

template <int KIND, RowsAt XL, bool YT>
static sl_status launch_split_kind(const LinearArgs &a, const GeluArg *ep, int wpw, hipStream_t stream)
{
    static_assert(kSplitWin == 2, "one instance per windows-per-wave count");
    if (wpw == 1) return launch_split_wpw<KIND, 1, XL, YT>(a, ep, stream);
    return launch_split_wpw<KIND, 2, XL, YT>(a, ep, stream);
}

template <int KIND, RowsAt XL>
static sl_status launch_split_y(const LinearArgs &a, const GeluArg *ep, int wpw, bool yt, hipStream_t stream)
{
    if constexpr (EpiOut<KIND>::kBytes == 1)
        if (yt) return launch_split_kind<KIND, XL, true>(a, ep, wpw, stream);
    return launch_split_kind<KIND, XL, false>(a, ep, wpw, stream);
}

template <int KIND>
static sl_status launch_split_x(const LinearArgs &a, const GeluArg *ep, int wpw, RowsAt xl, bool yt,
                                hipStream_t stream)
{
    switch (xl) {
    case RowsAt::kBlocks: return launch_split_y<KIND, RowsAt::kBlocks>(a, ep, wpw, yt, stream);
    case RowsAt::kWords: return launch_split_y<KIND, RowsAt::kWords>(a, ep, wpw, yt, stream);
    default: return launch_split_y<KIND, RowsAt::kBytes>(a, ep, wpw, yt, stream);
    }
}

int split_windows_per_wave(int32_t n_win)
{
    for (int wpw = 1; wpw <= kSplitWin; wpw *= 2)
        if (n_win <= wpw * kSplitMaxWaves) return wpw;
    return 0;
}

sl_status launch_split(const LinearArgs &a, const GeluArg *ep, int32_t run_kind, RowsAt xl, bool yt,
                       hipStream_t stream)
{
    const int wpw = split_windows_per_wave(a.n_win);
    if (wpw == 0 || a.kw < 1 || a.kw > kSplitMaxWaves || (int64_t)a.kw * wpw < a.n_win ||
        a.n_items > 0x7fffffff) {
        set_error("internal: split-reduction launch out of range");
        return SL_ERR_UNSUPPORTED;
    }
    if (a.n_items == 0) return SL_OK;
    switch (run_kind) {
    case SL_EPI_ACC_I32: return launch_split_x<SL_EPI_ACC_I32>(a, nullptr, wpw, xl, yt, stream);
    case SL_EPI_F32: return launch_split_x<SL_EPI_F32>(a, nullptr, wpw, xl, yt, stream);
    case SL_EPI_F32_GELU: return launch_split_x<SL_EPI_F32_GELU>(a, nullptr, wpw, xl, yt, stream);
    case SL_EPI_I8: return launch_split_x<SL_EPI_I8>(a, nullptr, wpw, xl, yt, stream);
    case SL_EPI_I8_GELU: return launch_split_x<SL_EPI_I8_GELU>(a, ep, wpw, xl, yt, stream);
    default: return launch_split_x<kEpiI8GeluErf>(a, nullptr, wpw, xl, yt, stream);
    }
}

}  // namespace sl

// The tile kernel of the sparse INT8 linear layer (gfx950): for long
// reductions over many tokens, with token rows in the block layout or
// row-major and 16-byte aligned.
//
// Same product as the other kernels (Section "Sparse GEMM operators", Figure
// 1, Algorithm 1), from the dense operand image (see kernels_panel.hip). A
// workgroup owns one tile of 128 tokens x NT 16-channel tiles and walks the
// reduction in 128-column windows: token rows and weight operands of a window
// are copied global to LDS (no registers) into a ring of D buffers, D - 1
// windows ahead. Its 8 waves are 2 along the tokens x 2 along the channels x
// 2 along the window: a wave multiplies 64 tokens x NT/2 tiles over one half
// of every window, which takes 4 + NT/2 LDS reads for 2 NT matrix instructions
// (32 tokens over whole windows would take 4 + NT). The two halves' int32 sums
// meet in LDS once at the end (exact in any order), and the finished tile goes
// out from there in whole rows.
//
// What bounds it: LDS (56 KB of operand reads and 28 KB of copies a window of a
// CU) and the copies' bytes from L2, with one barrier a window: about 890
// cycles a window against 405 of matrix instructions. It stands where the
// direct kernel's row loads touch 16 rows an instruction or its items need a
// round more (rules and figures at choose_tile_nt).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sl_device.h"

namespace sl {

template <int NT, int D>
struct TShape {
    static constexpr int TM = kTileTokens, TN = 16 * NT, CT = NT / 2;
    static constexpr int XC = TM / 8;       // 1024-byte copies of a window's token rows
    static constexpr int NCOPY = XC + 2 * NT;
    static constexpr int BUF = NCOPY * 1024;
    static constexpr int P4 = TN * 4 + 16;  // bytes between rows of the finished tile in LDS
    static constexpr int P1 = TN + 16;      // (int8 outputs)
    static constexpr int RING = D * BUF;
    static constexpr int VEC = 2 * TN * 4;  // scales sx * sw[n], then biases
    static_assert(TM * (P4 + P1) <= RING, "the finished tile takes the ring's place");
};

template <int KIND, int NT, int D, bool XT, bool YT>
__device__ __forceinline__ void tile_body(const LinearArgs &a, const GeluArg *ep)
{
    using S = TShape<NT, D>;
    constexpr int CT = S::CT, EB = EpiOut<KIND>::kBytes;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];
    float *const vec = reinterpret_cast<float *>(smem + S::RING);
    GeluCell *const tab = reinterpret_cast<GeluCell *>(smem + S::RING + S::VEC);

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const int g = lane >> 4, t = lane & 15;
    const int kh = wave & 1, wn = (wave >> 1) & 1, wm = wave >> 2;

    // consecutive works of one XCD share their token rows
    const int32_t work = (int32_t)xcd_work_index(blockIdx.x, gridDim.x);
    const int32_t mt = work / a.n_cgroups;
    const int32_t cg = work - mt * a.n_cgroups;
    const int64_t m0 = (int64_t)mt * S::TM;
    const int32_t tile0 = cg * NT;

    // the set-up's loads come before the copies, so that waiting for them does
    // not wait for the whole ring
    [[maybe_unused]] float scale = 0.0f, bias = 0.0f;
    [[maybe_unused]] GeluCell cell{};
    if constexpr (KIND != SL_EPI_ACC_I32) {
        const int32_t ch = tile0 * kTileN + tid;
        if (tid < S::TN && ch < a.n) {
            scale = a.w_scale[ch];
            bias = a.bias[ch];
        }
    }
    static_assert(kGeluCells <= kTileThreads, "one table cell a thread");
    if constexpr (KIND == SL_EPI_I8_GELU)
        if (tid < ep->nc) cell = ep->cell[tid];

    // ---- copies: wave v issues copies v, v + 8, ... of every window; the
    // first two are token rows, the others weight operands
    const int64_t mpad = (a.m + 15) / 16 * 16;
    const int64_t xbytes = XT ? mpad / 16 * a.x_cb * 512 : a.m * a.k;
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
        (void *)a.x, 0, (int)std::min<int64_t>(xbytes, kMaxBufferBytes), kRsrcWord3);
    const __amdgpu_buffer_rsrc_t wr =
        __builtin_amdgcn_make_buffer_rsrc((void *)a.dense, 0, (int)a.dense_bytes, kRsrcWord3);
    constexpr int NI = (S::NCOPY + 7) / 8;         // copies of the waves that have most
    const bool most = wave < S::NCOPY - 8 * (NI - 1);
    uint32_t off[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int j = wave + 8 * i;
        if (i < 2) {
            if constexpr (XT) {
                // two of the four 512-byte blocks of a 16-token subtile; tokens
                // 8..15 have the halves of their 32 bytes swapped, so that the
                // B operand reads use every bank
                const int q = lane & 31, tt = q >> 1;
                const int64_t tb = m0 / 16 + j / 2;
                off[i] = tb * 16 < mpad ? (uint32_t)((tb * a.x_cb + 2 * (j & 1) + (lane >> 5)) * 512 + tt * 32 +
                                                     (((q & 1) ^ (tt >> 3)) * 16))
                                        : kOob;
            } else {
                const int r = 8 * j + (lane >> 3);
                off[i] = m0 + r < a.m ? (uint32_t)((m0 + r) * a.k) + (uint32_t)(((lane & 7) ^ row_swizzle(r)) * 16) : kOob;
            }
        } else {
            off[i] = (uint32_t)(tile0 * kDenseOp) + (uint32_t)((j - S::XC) * 1024 + lane * 16);
        }
    }
    const uint32_t wstride = (uint32_t)a.n_tiles * (uint32_t)kDenseOp;
    auto copy_window = [&](int buf) {
        int8_t *const b = smem + buf * S::BUF;
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            if (i < NI - 1 || most)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(i < 2 ? xr : wr, (lds_void *)(b + (wave + 8 * i) * 1024), 16,
                                                         off[i], 0, 0, 0);
            off[i] += i < 2 ? (XT ? 4 * 512 : kWin) : wstride;
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d)
        if (d < a.n_win) copy_window(d);

    // ---- set-up
    if constexpr (KIND != SL_EPI_ACC_I32) {
        if (tid < S::TN) {
            vec[tid] = a.sx * scale;
            vec[S::TN + tid] = bias;
        }
    }
    float hinv = 0.0f, eoff = 0.0f, cmax = 0.0f;
    if constexpr (KIND == SL_EPI_I8_GELU) {
        if (tid < ep->nc) tab[tid] = cell;
        hinv = ep->hinv;
        eoff = ep->off;
        cmax = kGeluBase + (float)(ep->nc - 1);
    }

    // ---- operands: lane's LDS offsets in a buffer
    uint32_t bo[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const int r = wm * 64 + s * 16 + t;
        bo[s] = XT ? (uint32_t)((wm * 4 + s) * 2048 + (2 * kh + (g >> 1)) * 512 + t * 32 + (((g & 1) ^ (t >> 3)) * 16))
                   : (uint32_t)(r * kWin + (((4 * kh + g) ^ row_swizzle(r)) * 16));
    }
    const uint32_t ao = (uint32_t)(S::XC * 1024 + (wn * CT * 2 + kh) * 1024 + lane * 16);
    struct Ops {
        i32x4 b[4], a[CT];
    };
    Ops ops[2];
    auto read_ops = [&](Ops &o, int buf) {
        const int8_t *const p = smem + buf * S::BUF;
#pragma unroll
        for (int s = 0; s < 4; ++s) o.b[s] = *reinterpret_cast<const i32x4 *>(p + bo[s]);
#pragma unroll
        for (int c = 0; c < CT; ++c) o.a[c] = *reinterpret_cast<const i32x4 *>(p + ao + c * 2048);
    };
    i32x4 acc[CT][4];
#pragma unroll
    for (int c = 0; c < CT; ++c)
#pragma unroll
        for (int s = 0; s < 4; ++s) acc[c][s] = i32x4{0, 0, 0, 0};

    // Step w: once window w + 1 has landed for every wave (the copies issued
    // after it stay in flight) and every wave has read window w's buffer (in
    // step w - 1), the copies of window w + D start into that buffer, window
    // w + 1's operands are read, and window w's are multiplied.
    int buf1 = 0;
    auto landed = [&](int w) {  // window w, with w + D - 2 the last one issued
        if (w + D - 2 < a.n_win) {
            if (most)
                wait_vmcnt_le<(D - 2) * NI>();
            else
                wait_vmcnt_le<(D - 2) * (S::NCOPY % 8 ? NI - 1 : NI)>();
        } else {
            wait_vmcnt_le<0>();
        }
    };
    auto step = [&](auto pp, int w, int buf) {
        constexpr int P = decltype(pp)::value;
        landed(w + 1);
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        if (w + D < a.n_win) copy_window(buf);
        buf1 = buf + 1 == D ? 0 : buf + 1;
        // (the last step reads a buffer of an earlier window: no use is made of it)
        read_ops(ops[P ^ 1], buf1);
#pragma unroll
        for (int c = 0; c < CT; ++c)
#pragma unroll
            for (int s = 0; s < 4; ++s)
                acc[c][s] = __builtin_amdgcn_mfma_i32_16x16x64_i8(ops[P].a[c], ops[P].b[s], acc[c][s], 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4 + CT; ++v) {
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 4 * CT, 0);
        // window w + 1's buffer is refilled after the next barrier
        wait_lgkm0();
    };
    // window 0: with D - 1 windows issued after it
    if (D - 1 < a.n_win) {
        if (most)
            wait_vmcnt_le<(D - 1) * NI>();
        else
            wait_vmcnt_le<(D - 1) * (S::NCOPY % 8 ? NI - 1 : NI)>();
    } else {
        wait_vmcnt_le<0>();
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read_ops(ops[0], 0);
    wait_lgkm0();
    int w = 0, buf = 0;
    for (; w + 2 <= a.n_win; w += 2) {
        step(std::integral_constant<int, 0>{}, w, buf);
        step(std::integral_constant<int, 1>{}, w + 1, buf1);
        buf = buf1;
    }
    if (w < a.n_win) step(std::integral_constant<int, 0>{}, w, buf);

    // ---- the two halves of the reduction meet: wave kh finishes subtiles
    // 2 kh and 2 kh + 1 and hands the partial sums of the other two to its
    // partner
    __syncthreads();
    int8_t *const y4 = smem, *const y1 = smem + S::TM * S::P4;
    auto at4 = [&](int s, int c) { return y4 + (wm * 64 + s * 16 + t) * S::P4 + ((wn * CT + c) * 16 + 4 * g) * 4; };
    auto hand_over = [&](auto kk) {
        constexpr int OTHER = 2 * (1 - decltype(kk)::value);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int c = 0; c < CT; ++c) *reinterpret_cast<i32x4 *>(at4(OTHER + i, c)) = acc[c][OTHER + i];
    };
    auto finish = [&](auto kk) {
        constexpr int OWN = 2 * decltype(kk)::value;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
            float s4[4] = {0, 0, 0, 0}, b4[4] = {0, 0, 0, 0};
            if constexpr (KIND != SL_EPI_ACC_I32) {
                const int lc = (wn * CT + c) * 16 + 4 * g;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    s4[r] = vec[lc + r];
                    b4[r] = vec[S::TN + lc + r];
                }
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                i32x4 *const p = reinterpret_cast<i32x4 *>(at4(OWN + i, c));
                const auto o = epilogue_value<KIND>(a, *p + acc[c][OWN + i], s4, b4, tab, hinv, eoff, cmax);
                if constexpr (EB == 4)
                    *p = __builtin_bit_cast(i32x4, o);
                else
                    *reinterpret_cast<uint32_t *>(y1 + (wm * 64 + (OWN + i) * 16 + t) * S::P1 + (wn * CT + c) * 16 +
                                                  4 * g) = o;
            }
        }
    };
    using K0 = std::integral_constant<int, 0>;
    using K1 = std::integral_constant<int, 1>;
    if (kh)
        hand_over(K1{});
    else
        hand_over(K0{});
    __syncthreads();
    if (kh)
        finish(K1{});
    else
        finish(K0{});
    __syncthreads();
    // ---- the finished tile, 16 bytes a lane along its rows
    constexpr int PIECES = S::TN * EB / 16;
    int8_t *const y8 = static_cast<int8_t *>(a.y);
    const int64_t mlim = YT ? mpad : a.m;
    for (int u = tid; u < S::TM * PIECES; u += kTileThreads) {
        int r, p;
        if constexpr (YT) {
            // a 512-byte block of 16 tokens after the other
            const int b = u >> 5, q = u & 31;
            r = b / (S::TN / 32) * 16 + (q >> 1);
            p = b % (S::TN / 32) * 2 + (q & 1);
        } else {
            r = u / PIECES;
            p = u % PIECES;
        }
        const int64_t tok = m0 + r;
        const int32_t ch = tile0 * kTileN + p * (16 / EB);
        if (tok >= mlim || ch >= a.n) continue;
        const i32x4 v = *reinterpret_cast<const i32x4 *>(EB == 4 ? y4 + r * S::P4 + p * 16 : y1 + r * S::P1 + p * 16);
        if constexpr (EB == 4) {
            store_nt(y8 + (tok * a.n + ch) * 4, v);
        } else {
            int8_t *const d = YT ? y8 + t16x32_offset(tok, ch, a.y_cb) : y8 + tok * a.n + ch;
            if (YT || ch + 16 <= a.n) {
                store_nt_at4(d, v);
            } else {
                for (int i = 0; i < 4; ++i)
                    if (ch + 4 * i < a.n) store_nt(d + 4 * i, (uint32_t)v[i]);
            }
        }
    }
}

template <int KIND, int NT, int D, bool XT, bool YT>
__global__ __launch_bounds__(kTileThreads) void sparse_linear_tile_kernel(LinearArgs a)
{
    tile_body<KIND, NT, D, XT, YT>(a, nullptr);
}

template <int NT, int D, bool XT, bool YT>
__global__ __launch_bounds__(kTileThreads) void sparse_linear_tile_gelu_kernel(LinearArgs a, GeluArg ep)
{
    tile_body<SL_EPI_I8_GELU, NT, D, XT, YT>(a, &ep);
}

template <int KIND, int NT, bool XT, bool YT>
static sl_status launch_tile_nt(const LinearArgs &a, const GeluArg *ep, hipStream_t stream)
{
    constexpr int D = NT == 6 ? 5 : 4;
    using S = TShape<NT, D>;
    const void *fn;
    if constexpr (KIND == SL_EPI_I8_GELU)
        fn = reinterpret_cast<const void *>(&sparse_linear_tile_gelu_kernel<NT, D, XT, YT>);
    else
        fn = reinterpret_cast<const void *>(&sparse_linear_tile_kernel<KIND, NT, D, XT, YT>);
    constexpr size_t lds = (size_t)S::RING + S::VEC + (KIND == SL_EPI_I8_GELU ? kGeluLds : 0);
    static_assert(lds <= kLdsMax, "workgroup shape exceeds LDS");
    static int raised[kMaxDevices] = {};  // per kernel instance and device: LDS limit raised
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) {
        set_error("device index beyond the supported range");
        return SL_ERR_UNSUPPORTED;
    }
    if (!raised[dev]) {
        HIP_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax));
        raised[dev] = 1;
    }
    if constexpr (KIND == SL_EPI_I8_GELU)
        hipLaunchKernelGGL((sparse_linear_tile_gelu_kernel<NT, D, XT, YT>), dim3((uint32_t)a.n_items), dim3(kTileThreads), lds,
                           stream, a, *ep);
    else
        hipLaunchKernelGGL((sparse_linear_tile_kernel<KIND, NT, D, XT, YT>), dim3((uint32_t)a.n_items), dim3(kTileThreads), lds,
                           stream, a);
    HIP_TRY(hipGetLastError());
    return SL_OK;
}

template <int KIND, bool XT, bool YT>
static sl_status launch_tile_l(const LinearArgs &a, const GeluArg *ep, int nt, hipStream_t stream)
{
    return nt == 8 ? launch_tile_nt<KIND, 8, XT, YT>(a, ep, stream) : launch_tile_nt<KIND, 6, XT, YT>(a, ep, stream);
}

template <int KIND>
static sl_status launch_tile_kind(const LinearArgs &a, const GeluArg *ep, int nt, bool xt, bool yt, hipStream_t stream)
{
    if constexpr (EpiOut<KIND>::kBytes == 1)
        if (yt)
            return xt ? launch_tile_l<KIND, true, true>(a, ep, nt, stream)
                      : launch_tile_l<KIND, false, true>(a, ep, nt, stream);
    return xt ? launch_tile_l<KIND, true, false>(a, ep, nt, stream)
              : launch_tile_l<KIND, false, false>(a, ep, nt, stream);
}

sl_status launch_tile(const LinearArgs &a, const GeluArg *ep, int32_t run_kind, int nt, bool xt, bool yt,
                      hipStream_t stream)
{
    if (a.n_items < 1 || a.n_items > kTileMaxItems || (nt != 6 && nt != 8)) {
        set_error("internal: tile launch out of range");
        return SL_ERR_UNSUPPORTED;
    }
    switch (run_kind) {
    case SL_EPI_ACC_I32: return launch_tile_kind<SL_EPI_ACC_I32>(a, nullptr, nt, xt, yt, stream);
    case SL_EPI_F32: return launch_tile_kind<SL_EPI_F32>(a, nullptr, nt, xt, yt, stream);
    case SL_EPI_F32_GELU: return launch_tile_kind<SL_EPI_F32_GELU>(a, nullptr, nt, xt, yt, stream);
    case SL_EPI_I8: return launch_tile_kind<SL_EPI_I8>(a, nullptr, nt, xt, yt, stream);
    case SL_EPI_I8_GELU: return launch_tile_kind<SL_EPI_I8_GELU>(a, ep, nt, xt, yt, stream);
    default: return launch_tile_kind<kEpiI8GeluErf>(a, nullptr, nt, xt, yt, stream);
    }
}

}  // namespace sl

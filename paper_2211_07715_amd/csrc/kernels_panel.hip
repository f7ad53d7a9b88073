// The weight-stationary kernel of the sparse INT8 linear layer (gfx950): for
// token rows in either layout and at any alignment, when a channel group's
// whole weight panel fits in LDS.
//
// Same product as the other kernels (Section "Sparse GEMM operators", Figure
// 1, Algorithm 1: int8 products of the stored weight blocks with the input
// columns their mask names, int32 accumulation, one fused epilogue per output
// after the whole reduction), from the dense operand image: the stored blocks
// at their places in A operands of v_mfma_i32_16x16x64_i8, zeros elsewhere.
// The 4:2-sparse form needs an overflow operand beside the main one in 37 %
// of the (tile, window) pairs at 90 % sparsity and in 97 % at 80 %, and a
// branch per pair costs more than it saves, so both were multiplied: the same
// matrix time as the dense operands, 6 % more bytes, two index reads a tile,
// and twice the vector issue slots (a matrix instruction takes 8.7 cycles of
// them from the other waves of its SIMD in the sparse form, 4.7 in the dense
// one, measured beside a wave of fused multiply-adds).
//
// A workgroup owns one channel group (NT 16-channel tiles) and one slice of
// the tokens. It copies the group's panel into LDS once (back-to-back copies,
// nothing read before them), then its waves work through the slice's token
// groups on their own: a wave loads its token rows (the B operands) straight
// into registers, R - 1 windows ahead, and reads the weight operands from the
// resident panel three ahead of the matrix instructions that use them. Past
// the one barrier that follows the panel copy and the set-up there is none,
// so one wave's epilogue overlaps the matrix instructions of the others, and
// the weight image is read from memory once per workgroup rather than once
// per token tile.
//
// What bounds it: each wave's chain of matrix instructions and then epilogue,
// with two or three waves a SIMD to overlap them (at 49152 tokens FFN1's
// matrix instructions take 55 of its 114 us at the 2.13 GHz it runs at; timing
// copies: without the epilogue's arithmetic 87, without the matrix instructions
// 94, without the cache misses of the token rows 110, without the output stores
// or the LDS reads of the weights 116 each, no faster). Measured, us,
// 4:2-sparse operands -> dense: 4096 tokens, blocks: FFN1 at 90 % 14.4 ->
// 12.6, QKV at 80 % 12.4 -> 10.7; 49152 tokens: FFN1 139 -> 110, QKV 99 -> 79.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "sl_device.h"

namespace sl {

template <int NT, int ST, int NWV>
struct PShape {
    static constexpr int NTH = 64 * NWV;
    static constexpr int TG = 16 * ST;             // tokens per group
    static constexpr int VEC = 2 * NT * kTileN * 4;  // the group's scales sx * sw[n], then its biases
    static constexpr int WB = NT * kDenseOp;         // panel bytes of one window
    static constexpr int WC = WB / 1024;             // 1024-byte copies of one window
    // per wave: 16 token rows of 32 four-byte outputs (two tiles), padded to
    // 36 words so that neither the writes nor the reads of the transpose meet
    // a bank twice in one pass
    static constexpr int TRW = 36;
    static constexpr int TR = 16 * TRW * 4;
    static_assert(NT % 2 == 0 && ST % 2 == 0, "the int8 store takes four fragments");
};

// int32 / fp32 outputs in rows go through a per-wave LDS transpose
template <int KIND, bool YT, int NT>
constexpr bool panel_transposes()
{
    return NT % 2 == 0 && EpiOut<KIND>::kBytes == 4 && KIND != SL_EPI_F32_GELU && !YT;
}

// Row-major token rows change lanes through LDS for 4-byte outputs (us, without
// -> with: int32 QKV at 2048 tokens 10.2 -> 9.3, fp32 GELU FFN1 at 3072 20.1 ->
// 18.5); with int8 outputs, whose waves spend less on stores and more on
// arithmetic, the extra LDS steps cost as much as they save or more (FFN1 at
// 4096 17.9 -> 18.3, BERT-large FFN1 at 49152 222 -> 240).
template <int KIND, RowsAt XL>
using PanelRows = RowSource<XL, XL == RowsAt::kWords && EpiOut<KIND>::kBytes == 4>;

// LDS layout: weight scales and biases | GELU step table | per-wave areas (the
// transpose, and token rows that change lanes) | panel
template <int KIND, int NT, int ST, int NWV, RowsAt XL, bool YT>
struct PLds {
    using S = PShape<NT, ST, NWV>;
    static constexpr int kTab = KIND == SL_EPI_I8_GELU ? kGeluLds : 0;
    static constexpr int kWave = std::max(panel_transposes<KIND, YT, NT>() ? S::TR : 0, PanelRows<KIND, XL>::kScratch);
    static constexpr int kFixed = S::VEC + kTab + NWV * kWave;
    static_assert(kFixed % 256 == 0 && S::WB % 256 == 0, "16-byte copies; the table of resident workgroups");
    static size_t bytes(uint64_t panel) { return (size_t)kFixed + panel; }
};

// Calls f(std::integral_constant<int, 0>) .. f(std::integral_constant<int, N-1>) in order.
template <int... Us, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, Us...>, F &&f)
{
    (f(std::integral_constant<int, Us>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// R: windows of token rows held in registers (R - 1 of them loading while
// one is multiplied)
// XL: where the token rows lie (RowsAt).
template <int KIND, int NT, int ST, int NWV, int R, RowsAt XL, bool YT>
__device__ __forceinline__ void panel_body(const LinearArgs &a, const GeluArg *ep)
{
    using S = PShape<NT, ST, NWV>;
    using L = PLds<KIND, NT, ST, NWV, XL, YT>;
    extern __shared__ __attribute__((aligned(16))) int8_t smem[];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;

    // work: channel group cg, token slice ts; the workgroups of one XCD take
    // consecutive works, which share a token slice
    const int32_t work = (int32_t)xcd_work_index(blockIdx.x, gridDim.x);
    const int32_t ts = work / a.n_cgroups;
    const int32_t cg = work - ts * a.n_cgroups;
    const int32_t tile0 = cg * NT;

    float *const vec = reinterpret_cast<float *>(smem);
    GeluCell *const tab = reinterpret_cast<GeluCell *>(smem + S::VEC);
    int8_t *const trans = smem + S::VEC + L::kTab + wave * L::kWave;
    int8_t *const panel = smem + L::kFixed;

    // ---- the group's panel: [window][tile] pairs of operands, copied global
    // to LDS (no registers) in 1024-byte instructions, wave v issuing
    // instructions v, v + NWV, ...; nothing is read before them, so the copies
    // start at once and land while the set-up runs. (Tiles past the last one
    // read the next window's, or zeros past the image: their channels are
    // never stored.)
    {
        constexpr int kMaxCopies = (int)((kLdsMax / 1024 + NWV - 1) / NWV);
        const __amdgpu_buffer_rsrc_t ir =
            __builtin_amdgcn_make_buffer_rsrc((void *)a.dense, 0, (int)a.dense_bytes, kRsrcWord3);
        const uint32_t src = (uint32_t)tile0 * kDenseOp + (uint32_t)lane * 16u;
        const uint32_t wstride = (uint32_t)a.n_tiles * kDenseOp;
        const int n_copies = a.n_win * S::WC;
#pragma unroll
        for (int i = 0; i < kMaxCopies; ++i) {
            const int j = wave + i * NWV;
            if (j < n_copies)
                __builtin_amdgcn_raw_ptr_buffer_load_lds(
                    ir, (lds_void *)(panel + (size_t)j * 1024), 16,
                    src + (uint32_t)(j / S::WC) * wstride + (uint32_t)(j % S::WC) * 1024u, 0, 0, 0);
        }
    }

    float hinv = 0.0f, eoff = 0.0f, cmax = 0.0f;  // GELU table parameters (set-up below)

    // ---- token groups of this workgroup's slice, one wave each at a time
    const int64_t mpad = (a.m + 15) / 16 * 16;
    const int64_t slice0 = (int64_t)ts * a.slice_groups * S::TG;
    const int n_groups = (int)std::min<int64_t>(a.slice_groups, (mpad - slice0 + S::TG - 1) / S::TG);

    const PanelRows<KIND, XL> src(a);
    // Token rows: lane l of subtile s loads features 16*(l/16) .. +15 of each
    // half of the window for token (l % 16) -- the B operand layout. Tokens past m read
    // zeros (out-of-range offsets) or a padding token of the last block; a
    // ragged last window reads bytes past the row (or zeros past the buffer),
    // which meet zero weights.
    auto row_offsets = [&](int64_t t0, uint32_t (&ro)[ST]) {
#pragma unroll
        for (int s = 0; s < ST; ++s) ro[s] = src.offset(a, t0 + s * 16 + src.load_token(lane), src.load_group(lane));
    };
    auto load_rows = [&](RowPiece<XL> (&bv)[ST], const uint32_t (&ro)[ST], int w) {
#pragma unroll
        for (int s = 0; s < ST; ++s) bv[s] = src.load(ro[s], w);
    };

    i32x4 acc[NT][ST];
    RowPiece<XL> bv[R][ST];
    static_assert(R >= 2, "at least one window loads while another is multiplied");

    // Weight operands in registers, a ring of RS units (one half-window of one
    // tile each) filled LA units ahead of the matrix instructions: while unit
    // c of window u is multiplied, unit c + LA of the wave's stream is read
    // (of window u, else of window u + 1; past the group's last window that
    // is the first window of the next group, which uses the same panel). RS
    // divides the units of a window, so a unit's slot is c % RS.
    constexpr int NU = 2 * NT;
    constexpr int RS = 4;
    constexpr int LA = RS - 1;
    static_assert(NU % RS == 0 && LA >= 1, "ring slots follow from the unit");
    i32x4 ring[RS];
    auto read_unit = [&](i32x4 &t, uint32_t base, int c) {
        t = *reinterpret_cast<const i32x4 *>(panel + base + (2 * (c % NT) + c / NT) * 1024 + lane * 16);
    };
    // window u (token rows in ring slot PB, panel bytes cbase; the next
    // window's at nbase)
    // (ro: the group's row offsets, whose low bits say how its rows lie)
    auto multiply = [&](auto pb, uint32_t cbase, uint32_t nbase, const uint32_t (&ro)[ST]) {
        constexpr int PB = decltype(pb)::value;
        i32x4 rows[2][ST];
#pragma unroll
        for (int s = 0; s < ST; ++s) {
            rows[0][s] = src.operand(bv[PB][s], 0, ro[s], trans, lane);
            rows[1][s] = src.operand(bv[PB][s], 1, ro[s], trans, lane);
        }
        static_for<NU>([&](auto cc) {
            constexpr int C = decltype(cc)::value;
            constexpr int J = C + LA;
            if constexpr (J < NU)
                read_unit(ring[J % RS], cbase, J);
            else
                read_unit(ring[J % RS], nbase, J - NU);
#pragma unroll
            for (int s = 0; s < ST; ++s)
                acc[C % NT][s] =
                    __builtin_amdgcn_mfma_i32_16x16x64_i8(ring[C % RS], rows[C / NT][s], acc[C % NT][s], 0, 0, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // one LDS read
            __builtin_amdgcn_sched_group_barrier(0x008, ST, 0);  // its matrix instructions
        });
    };

    // Int8 epilogues whose temporaries of two fragments do not fit beside the
    // accumulators finish one fragment before the next begins: erf's, and the
    // table's in the 168 registers of 12 waves with 8 tiles or with row
    // addresses. Left to the scheduler they spilled 28 to 200 bytes a lane; us,
    // two fragments -> one: erf, FFN1 768 -> 3072 in blocks at 4096 / 49152
    // tokens 26.7 -> 20.6 / 228 -> 211; table, 1024 -> 4096 in blocks at 2048 /
    // 4096 / 49152 tokens 18.8 -> 15.0 / 25.3 -> 22.8 / 198 -> 183.
    constexpr bool kOneFragment =
        KIND == kEpiI8GeluErf || (KIND == SL_EPI_I8_GELU && NWV == 12 && (NT == 8 || !YT));
    // accumulator layout: lane l holds rows 4*(l/16)+r (channels of one
    // block-row), column l%16 (token), r = 0..3
    auto scales = [&](int c, float (&s)[4], float (&bb4)[4]) {
        if constexpr (KIND != SL_EPI_ACC_I32) {
            const int lc = c * kTileN + 4 * (lane >> 4);
            const float4 sw = *reinterpret_cast<const float4 *>(vec + lc);
            const float4 bb = *reinterpret_cast<const float4 *>(vec + NT * kTileN + lc);
            s[0] = sw.x;
            s[1] = sw.y;
            s[2] = sw.z;
            s[3] = sw.w;
            bb4[0] = bb.x;
            bb4[1] = bb.y;
            bb4[2] = bb.z;
            bb4[3] = bb.w;
        } else {
            for (int r = 0; r < 4; ++r) s[r] = bb4[r] = 0.0f;
        }
    };
    auto epilogue = [&](int64_t t0) {
        // in the block layout the padding tokens of the last block may be
        // written too
        const int64_t mlim = YT ? mpad : a.m;
        const bool whole = t0 + S::TG <= mlim && (tile0 + NT) * kTileN <= a.n;
        if constexpr (EpiOut<KIND>::kBytes == 1) {
            if (whole) {
                // int8 codes: a lane holds 4 channels of one token, and four
                // fragments (a tile of a subtile each) are transposed across
                // the four lane groups in registers, after which lane group g
                // holds the 16 channels of fragment g: 16 contiguous bytes a
                // lane, in either layout.
                int8_t *const y8 = static_cast<int8_t *>(a.y);
                const int g = lane >> 4, t = lane & 15;
                // fragments: four tiles of one subtile, or (Q) two tiles of two
                auto quad = [&](auto c0, auto s0, auto two) {
                    constexpr int C0 = decltype(c0)::value, S0 = decltype(s0)::value;
                    constexpr bool Q = decltype(two)::value;
                    uint32_t v[4];
                    // (two fragments at a time: the GELU kind's table reads
                    // of 8 outputs a lane are in flight together; one at a
                    // time where two do not fit in registers)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const int ca = C0 + (Q ? 0 : 2 * h), sa = S0 + (Q ? h : 0);
                        float s0[4], b0[4], s1[4], b1[4];
                        scales(ca, s0, b0);
                        scales(ca + 1, s1, b1);
                        if constexpr (KIND == SL_EPI_I8_GELU && !kOneFragment) {
                            float gy[2][4];
                            uint32_t ad[2][4];
                            u32x2 cell[2][4];
                            gelu_cells(acc[ca][sa], s0, b0, tab, hinv, eoff, cmax, gy[0], ad[0]);
                            gelu_cells(acc[ca + 1][sa], s1, b1, tab, hinv, eoff, cmax, gy[1], ad[1]);
#pragma unroll
                            for (int j = 0; j < 2; ++j)
#pragma unroll
                                for (int r = 0; r < 4; ++r) cell[j][r] = lds_read_u2(ad[j][r]);
                            v[2 * h] = gelu_codes(gy[0], cell[0]);
                            v[2 * h + 1] = gelu_codes(gy[1], cell[1]);
                        } else {
                            v[2 * h] = epilogue_value<KIND>(a, acc[ca][sa], s0, b0, tab, hinv, eoff, cmax);
                            if constexpr (kOneFragment) __builtin_amdgcn_sched_barrier(0);
                            v[2 * h + 1] = epilogue_value<KIND>(a, acc[ca + 1][sa], s1, b1, tab, hinv, eoff, cmax);
                            if constexpr (kOneFragment) __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                    transpose4(v);
                    int8_t *p;
                    if constexpr (YT)
                        p = y8 + ((t0 / 16 + S0) * a.y_cb + (tile0 + C0) / 2) * 512 +
                            (uint32_t)((g >> 1) * (Q ? a.y_cb * 512 : 512) + t * 32 + (g & 1) * 16);
                    else
                        p = y8 + (t0 + S0 * 16) * a.n + (tile0 + C0) * kTileN +
                            (uint32_t)((t + (Q ? (g >> 1) * 16 : 0)) * a.n + (Q ? g & 1 : g) * 16);
                    // (rows of Y start at multiples of 4 bytes)
                    store_nt_at4(p, i32x4{(int)v[0], (int)v[1], (int)v[2], (int)v[3]});
                };
                static_for<NT / 4>([&](auto cq) {
                    static_for<ST>([&](auto sq) {
                        quad(std::integral_constant<int, 4 * decltype(cq)::value>{}, sq, std::false_type{});
                    });
                });
                if constexpr (NT % 4 != 0)
                    static_for<ST / 2>([&](auto sq) {
                        quad(std::integral_constant<int, NT / 4 * 4>{},
                             std::integral_constant<int, 2 * decltype(sq)::value>{}, std::true_type{});
                    });
                return;
            }
        } else if constexpr (panel_transposes<KIND, YT, NT>()) {
            if (whole) {
                // a lane's 16 bytes sit in a different row from its quad
                // neighbours', so each pair of tiles goes through this wave's
                // LDS transpose area; a store then writes 8 tokens x 32
                // channels (128 contiguous bytes a token, 8 lanes a row)
                int32_t *const tr = reinterpret_cast<int32_t *>(trans);
                const int wi = (lane & 15) * S::TRW + 4 * (lane >> 4);  // write: token l%16, channels 4(l/16)..
                const int ri = (lane >> 3) * S::TRW + 4 * (lane & 7);   // read: token l/8 (+8), channels 4(l%8)..
                int8_t *const y8 = static_cast<int8_t *>(a.y);
#pragma unroll
                for (int c = 0; c < NT; c += 2) {
                    float s0[4], b0[4], s1[4], b1[4];
                    scales(c, s0, b0);
                    scales(c + 1, s1, b1);
#pragma unroll
                    for (int st = 0; st < ST; ++st) {
                        const i32x4 v0 = __builtin_bit_cast(
                            i32x4, epilogue_value<KIND>(a, acc[c][st], s0, b0, tab, hinv, eoff, cmax));
                        const i32x4 v1 = __builtin_bit_cast(
                            i32x4, epilogue_value<KIND>(a, acc[c + 1][st], s1, b1, tab, hinv, eoff, cmax));
                        // (a wave's LDS operations take effect in order: the
                        // previous pair's reads are done before these writes)
                        *reinterpret_cast<i32x4 *>(tr + wi) = v0;
                        *reinterpret_cast<i32x4 *>(tr + wi + 16) = v1;
                        const i32x4 r0 = *reinterpret_cast<const i32x4 *>(tr + ri);
                        const i32x4 r1 = *reinterpret_cast<const i32x4 *>(tr + ri + 8 * S::TRW);
                        const int64_t row = t0 + st * 16 + (lane >> 3);
                        int8_t *const p = y8 + (row * a.n + (tile0 + c) * kTileN + 4 * (lane & 7)) * 4;
                        store_nt(p, r0);
                        store_nt(p + (int64_t)8 * a.n * 4, r1);
                    }
                }
                return;
            }
        }
        if (whole) {
            // whole group: a uniform base and a lane offset, no bounds checks
            constexpr int EB = EpiOut<KIND>::kBytes;
            int8_t *const y8 = static_cast<int8_t *>(a.y);
            const uint32_t lo = YT ? (uint32_t)(32 * (lane & 15) + 4 * (lane >> 4))
                                   : (uint32_t)(((lane & 15) * a.n + 4 * (lane >> 4)) * EB);
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                float s[4], bb4[4];
                scales(c, s, bb4);
#pragma unroll
                for (int st = 0; st < ST; ++st) {
                    const int32_t ch = (tile0 + c) * kTileN;
                    const int64_t uo =
                        YT ? t16x32_offset(t0 + st * 16, ch, a.y_cb) : ((t0 + st * 16) * a.n + ch) * EB;
                    store_nt(y8 + uo + lo, epilogue_value<KIND>(a, acc[c][st], s, bb4, tab, hinv, eoff, cmax));
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < NT; ++c) {
                const int32_t t = tile0 + c;
                if (t >= a.n_tiles) break;
                const int32_t ch0 = t * kTileN + 4 * (lane >> 4);
                if (ch0 >= a.n) continue;  // block-rows past n_out in the last tile
                float s[4], bb4[4];
                scales(c, s, bb4);
#pragma unroll
                for (int st = 0; st < ST; ++st)
                    epilogue_store<KIND, YT>(a, acc[c][st], t0 + st * 16 + (lane & 15), ch0, s, bb4, tab, hinv,
                                             eoff, cmax);
            }
        }
    };

    // The wave's (token group, window) elements form one stream: groups
    // wave, wave + NWV, ... of the slice, each padded to whole turns of the
    // R-window ring, so the u-th window of every group uses ring slot u % R.
    // Before multiplying element e the wave starts loading element e + R - 1
    // (possibly a window of its next group), so the next group's first
    // windows load during the current group's epilogue. (Starting each
    // workgroup and wave at a group and window of its own, so that those that
    // share token rows read them at different times, changes nothing.)
    const int n_my = n_groups > wave ? (n_groups - wave + NWV - 1) / NWV : 0;
    const int nwp = (a.n_win + R - 1) / R * R;
    auto group_t0 = [&](int i) {
        return slice0 + (int64_t)(wave + i * NWV) * S::TG;
    };
    uint32_t ro[ST], ron[ST];
    // panel byte of window u
    auto wbase = [&](int u) { return (uint32_t)u * (uint32_t)S::WB; };
    // the first R - 1 windows of token rows load while the panel copies are
    // in flight, then the set-up; one barrier after all of them, past which
    // table, panel, scales and GELU table are in LDS
    row_offsets(n_my > 0 ? group_t0(0) : slice0, ro);
    static_for<R - 1>([&](auto uc) {
        constexpr int U = decltype(uc)::value;
        load_rows(bv[U], ro, U);
    });
    // ---- set-up: scales and biases, GELU table
    static_assert(NT * kTileN <= S::NTH, "one scale and one bias a thread");
    if constexpr (KIND != SL_EPI_ACC_I32) {
        if (tid < NT * kTileN) {
            const int32_t ch = tile0 * kTileN + tid;
            // the dequantisation scale sx * sw[n], one fp32 product as in the definition
            vec[tid] = ch < a.n ? a.sx * a.w_scale[ch] : 0.0f;
            vec[NT * kTileN + tid] = ch < a.n ? a.bias[ch] : 0.0f;
        }
    }
    if constexpr (KIND == SL_EPI_I8_GELU) {
        for (int u = tid; u < ep->nc; u += S::NTH) tab[u] = ep->cell[u];
        hinv = ep->hinv;
        eoff = ep->off;
        cmax = kGeluBase + (float)(ep->nc - 1);
    }
    // every wave's copies (and first token rows) have landed before the barrier
    wait_vmcnt_le<0>();
    __syncthreads();
    if (n_my > 0) {
#pragma unroll
        for (int j = 0; j < LA; ++j) read_unit(ring[j], wbase(0), j);
    }
    for (int i = 0; i < n_my; ++i) {
        const int64_t t0 = group_t0(i);
        const bool has_next = i + 1 < n_my;
        row_offsets(has_next ? group_t0(i + 1) : mpad, ron);
#pragma unroll
        for (int c = 0; c < NT; ++c)
#pragma unroll
            for (int s = 0; s < ST; ++s) acc[c][s] = i32x4{0, 0, 0, 0};
        for (int wb = 0; wb < nwp; wb += R) {
            static_for<R>([&](auto uc) {
                constexpr int U = decltype(uc)::value;
                constexpr int PS = (U + R - 1) % R;
                const int u = wb + U;
                const int pu = u + R - 1;
                // past the group's windows: the next group's (rows past the
                // last group read zeros)
                const bool in_cur = pu < nwp;
                uint32_t rs[ST];
#pragma unroll
                for (int s = 0; s < ST; ++s) rs[s] = in_cur ? ro[s] : ron[s];
                load_rows(bv[PS], rs, in_cur ? pu : pu - nwp);
                if (u < a.n_win) {
                    // the ring reads ahead into this group's next window,
                    // else the next group's first (a stale read past the
                    // last group)
                    multiply(uc, wbase(u), wbase(u + 1 < a.n_win ? u + 1 : 0), ro);
                }
            });
        }
        epilogue(t0);
        if (has_next) {
#pragma unroll
            for (int s = 0; s < ST; ++s) ro[s] = ron[s];
        }
    }
}

template <int KIND, int NT, int ST, int NWV, int R, RowsAt XL, bool YT>
__global__ __launch_bounds__(64 * NWV) void sparse_linear_panel_kernel(LinearArgs a)
{
    panel_body<KIND, NT, ST, NWV, R, XL, YT>(a, nullptr);
}

template <int NT, int ST, int NWV, int R, RowsAt XL, bool YT>
__global__ __launch_bounds__(64 * NWV) void sparse_linear_panel_gelu_kernel(LinearArgs a, GeluArg ep)
{
    panel_body<SL_EPI_I8_GELU, NT, ST, NWV, R, XL, YT>(a, &ep);
}

template <int KIND, int NT, int ST, int NWV, int R, RowsAt XL, bool YT>
static const void *panel_fn()
{
    if constexpr (KIND == SL_EPI_I8_GELU)
        return reinterpret_cast<const void *>(&sparse_linear_panel_gelu_kernel<NT, ST, NWV, R, XL, YT>);
    else
        return reinterpret_cast<const void *>(&sparse_linear_panel_kernel<KIND, NT, ST, NWV, R, XL, YT>);
}

template <int KIND, int NT, int ST, int NWV, int R, RowsAt XL, bool YT>
static sl_status launch_panel_cfg(const LinearArgs &a, const GeluArg *ep, size_t lds, hipStream_t stream)
{
    using S = PShape<NT, ST, NWV>;
    const void *fn = panel_fn<KIND, NT, ST, NWV, R, XL, YT>();
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
    const int64_t nwg = (int64_t)a.n_cgroups * a.n_slices;
    if constexpr (KIND == SL_EPI_I8_GELU)
        hipLaunchKernelGGL((sparse_linear_panel_gelu_kernel<NT, ST, NWV, R, XL, YT>), dim3((uint32_t)nwg),
                           dim3(S::NTH), lds, stream, a, *ep);
    else
        hipLaunchKernelGGL((sparse_linear_panel_kernel<KIND, NT, ST, NWV, R, XL, YT>), dim3((uint32_t)nwg),
                           dim3(S::NTH), lds, stream, a);
    HIP_TRY(hipGetLastError());
    return SL_OK;
}

// The compiled shapes: F(NT, ST, NWV, R).
#define SL_PANEL_SHAPES(F) \
    F(6, 2, 12, 2)         \
    F(6, 2, 8, 2)          \
    F(4, 2, 8, 2)          \
    F(2, 2, 8, 4)          \
    F(2, 4, 4, 2)          \
    F(8, 2, 8, 2)          \
    F(8, 2, 12, 2)

const PanelCfg kPanelCfgs[kNumPanelCfgs] = {
#define SL_PANEL_ENTRY(NT_, ST_, NWV_, R_) {NT_, ST_, NWV_, R_},
    SL_PANEL_SHAPES(SL_PANEL_ENTRY)
#undef SL_PANEL_ENTRY
};

template <int KIND, RowsAt XL, bool YT>
static sl_status launch_panel_kind(const LinearArgs &a, const GeluArg *ep, PanelCfg c, size_t lds,
                                   hipStream_t stream)
{
#define SL_PANEL_CASE(NT_, ST_, NWV_, R_)                                \
    if constexpr (XL != RowsAt::kBytes || panel_takes_bytes(NT_, ST_, NWV_, R_))            \
        if (c.nt == NT_ && c.st == ST_ && c.nwv == NWV_ && c.r == R_)                       \
            return launch_panel_cfg<KIND, NT_, ST_, NWV_, R_, XL, YT>(a, ep, lds, stream);
    SL_PANEL_SHAPES(SL_PANEL_CASE)
#undef SL_PANEL_CASE
    set_error("internal: unknown weight-stationary workgroup shape");
    return SL_ERR_UNSUPPORTED;
}

template <int KIND, RowsAt XL, bool YT>
static size_t panel_lds_shape(PanelCfg c, uint64_t panel)
{
#define SL_PANEL_LDS(NT_, ST_, NWV_, R_)                          \
    if (c.nt == NT_ && c.st == ST_ && c.nwv == NWV_ && c.r == R_) \
        return PLds<KIND, NT_, ST_, NWV_, XL, YT>::bytes(panel);
    SL_PANEL_SHAPES(SL_PANEL_LDS)
#undef SL_PANEL_LDS
    return (size_t)-1;
}

template <int KIND, bool YT>
static size_t panel_lds_kind(PanelCfg c, RowsAt xl, uint64_t panel)
{
    // (blocks and rows at any byte take the same)
    return xl == RowsAt::kWords ? panel_lds_shape<KIND, RowsAt::kWords, YT>(c, panel)
                                : panel_lds_shape<KIND, RowsAt::kBlocks, YT>(c, panel);
}

size_t panel_lds_bytes(PanelCfg c, int32_t run_kind, RowsAt xl, bool yt, uint64_t panel)
{
    switch (run_kind) {
    case SL_EPI_ACC_I32: return panel_lds_kind<SL_EPI_ACC_I32, false>(c, xl, panel);
    case SL_EPI_F32: return panel_lds_kind<SL_EPI_F32, false>(c, xl, panel);
    case SL_EPI_F32_GELU: return panel_lds_kind<SL_EPI_F32_GELU, false>(c, xl, panel);
    case SL_EPI_I8_GELU:
        return yt ? panel_lds_kind<SL_EPI_I8_GELU, true>(c, xl, panel)
                  : panel_lds_kind<SL_EPI_I8_GELU, false>(c, xl, panel);
    default:  // SL_EPI_I8, and with erf
        return yt ? panel_lds_kind<SL_EPI_I8, true>(c, xl, panel) : panel_lds_kind<SL_EPI_I8, false>(c, xl, panel);
    }
}

sl_status panel_resident(PanelCfg c, size_t lds, int *out)
{
    const void *fn = nullptr;
    int threads = 0;
#define SL_PANEL_FN(NT_, ST_, NWV_, R_)                                          \
    if (c.nt == NT_ && c.st == ST_ && c.nwv == NWV_ && c.r == R_) {              \
        fn = panel_fn<SL_EPI_F32, NT_, ST_, NWV_, R_, RowsAt::kBlocks, false>();            \
        threads = PShape<NT_, ST_, NWV_>::NTH;                                   \
    }
    SL_PANEL_SHAPES(SL_PANEL_FN)
#undef SL_PANEL_FN
    if (!fn) {
        set_error("internal: unknown weight-stationary workgroup shape");
        return SL_ERR_UNSUPPORTED;
    }
    int dev = 0, per_cu = 0, n_cu = 0;
    HIP_TRY(hipGetDevice(&dev));
    HIP_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLdsMax));
    HIP_TRY(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev));
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, threads, lds));
    *out = per_cu * n_cu;
    return SL_OK;
}

template <int KIND, RowsAt XL>
static sl_status launch_panel_y(const LinearArgs &a, const GeluArg *ep, PanelCfg c, bool yt, size_t lds,
                                hipStream_t stream)
{
    if constexpr (EpiOut<KIND>::kBytes == 1)
        if (yt) return launch_panel_kind<KIND, XL, true>(a, ep, c, lds, stream);
    return launch_panel_kind<KIND, XL, false>(a, ep, c, lds, stream);
}

template <int KIND>
static sl_status launch_panel_x(const LinearArgs &a, const GeluArg *ep, PanelCfg c, RowsAt xl, bool yt, size_t lds,
                                hipStream_t stream)
{
    switch (xl) {
    case RowsAt::kBlocks: return launch_panel_y<KIND, RowsAt::kBlocks>(a, ep, c, yt, lds, stream);
    case RowsAt::kWords: return launch_panel_y<KIND, RowsAt::kWords>(a, ep, c, yt, lds, stream);
    default: return launch_panel_y<KIND, RowsAt::kBytes>(a, ep, c, yt, lds, stream);
    }
}

sl_status launch_panel(const LinearArgs &a, const GeluArg *ep, int32_t run_kind, PanelCfg c, RowsAt xl, bool yt,
                       size_t lds, hipStream_t stream)
{
    switch (run_kind) {
    case SL_EPI_ACC_I32: return launch_panel_x<SL_EPI_ACC_I32>(a, nullptr, c, xl, yt, lds, stream);
    case SL_EPI_F32: return launch_panel_x<SL_EPI_F32>(a, nullptr, c, xl, yt, lds, stream);
    case SL_EPI_F32_GELU: return launch_panel_x<SL_EPI_F32_GELU>(a, nullptr, c, xl, yt, lds, stream);
    case SL_EPI_I8: return launch_panel_x<SL_EPI_I8>(a, nullptr, c, xl, yt, lds, stream);
    case SL_EPI_I8_GELU: return launch_panel_x<SL_EPI_I8_GELU>(a, ep, c, xl, yt, lds, stream);
    default: return launch_panel_x<kEpiI8GeluErf>(a, nullptr, c, xl, yt, lds, stream);
    }
}

}  // namespace sl

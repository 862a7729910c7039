// Flash Swin attention backward, fp32 storage and arithmetic, gfx950 (CDNA4) matrix cores, and
// the reduction of the pad token's gradient shared with the bf16 path.
//
// The gradients of Eq. 1 inside each window (the paper trains through Flash Swin, App. D),
// with c = 1/sqrt(d), LSE_i stored by the training forward and D_i = <dO_i, O_i>:
//   P_ij = w_j exp(c <q_i, k_j> - LSE_i),  dS_ij = P_ij (<dO_i, v_j> - D_i)
//   dq_i = c sum_j dS_ij k_j,   dk_j = c sum_i dS_ij q_i,   dv_j = sum_i P_ij dO_i
// Nothing of size n^2 is stored: P is recomputed from q, k and LSE.
//
// One launch, two kinds of workgroup (256 threads = 4 waves) per (batch entry, window, block of
// 64 tokens, head); wave (tt, sh) owns the 32 tokens of tile tt of the block and works on
// every other 32-row tile of what streams past (tiles sh, sh + 2, ...); the two waves of a tile
// add their sums at the end:
//   * key role: the K and V rows of its 32 keys in registers, the window's queries streaming
//     (Q, dO rows; LSE, D per query):   S = Q K_w^T, dP - D = dO V_w^T - D,
//     dV_w^T += dO^T P, dK_w^T += Q^T dS;
//   * query role: the Q and dO rows of its 32 queries in registers, the window's keys streaming:
//     S^T = K Q_w^T, dP^T - D = V dO_w^T - D, dQ_w^T += K^T dS^T.
// Products run on v_mfma_f32_32x32x2_f32, laid out as in the fp32 forward: the channel sums take
// half h = l / 32 of a row's channels per lane, 16 bytes of a streamed row at a time, and the
// accumulator of S (the streamed rows 8 (r / 4) + 4 h + r % 4 in register r) is, after the
// elementwise step, the second operand of the product summed over those rows, whose first
// operand is a 4-byte read of the streamed row.
//
// Streamed rows come 64 at a time by buffer loads that write LDS, into one of two buffers: the
// next chunk's loads are issued when a chunk is published, one barrier per chunk.  The 16-byte
// pieces of a row are XOR-swizzled by the row.  64 KB of row buffers and up to 256 VGPRs: two
// workgroups share a compute unit.
//
// Bound by the fp32 matrix rate (64 flop per cycle and SIMD): seven products of 32 x 64
// cycles per pair of 32-token tiles, against five if dS were shared between the roles; sharing
// it needs the whole window in one workgroup, which leaves most of the chip idle on the small
// grids that fp32 is used for.
// Measured, 12 heads, window 16, shift 8: 64x64 tokens 109 us, 128x128 432 us; three kernels of
// one token per thread on the vector ALU, the streamed rows broadcast from LDS, took 641 and
// 1708 us.
//
// KV-token mode: the pad token (Sec. 3.4, App. B) is one more key of weight n_pad.  The query role
// adds its dS_p k_p to dQ; the key role of block 0, past which every query of the window streams,
// sums the pad token's own gradient over them into the workspace, one partial per window.
// The pad reduce kernel then sums those in a fixed order into row L of dk and dv, so the
// result does not depend on scheduling.
#include "fla_swin_device.h"

namespace fla {
namespace {

constexpr int D = kHeadDim;
constexpr int THREADS = 256;
constexpr int NW = THREADS / 64;
constexpr int TL = 32;                 // tokens per tile
constexpr int TB = 2 * TL;             // tokens per block: two waves per tile
constexpr int CH = 2 * TL;             // streamed rows per chunk: one tile per sh
constexpr int ROWP = D / 4;            // 16-byte pieces per row
constexpr int BUF = CH * D;            // floats of one chunk's rows of one tensor
// log2(e) in two parts: LSE log2(e) is kept as a pair, so that P carries the rounding of the
// stored LSE and not that of a product of its size as well
constexpr float kLog2eHi = 1.44269502f, kLog2eLo = 1.92596303e-8f;

// LDS, floats: two buffers of X rows (Q or K) and Y rows (dO or V); per streamed query of each
// buffer LSE log2(e) (two parts), -D, and the pad token's P and dS; the pad token's k and v rows,
// and two half sums per channel of its gradient.  After the last chunk the row buffers hold the
// exchanged halves of the accumulators (OFF_EXCH) and the finished rows.
constexpr int OFF_X = 0;
constexpr int OFF_Y = OFF_X + 2 * BUF;
constexpr int OFF_LH = OFF_Y + 2 * BUF;
constexpr int OFF_LL = OFF_LH + 2 * CH;
constexpr int OFF_ND = OFF_LL + 2 * CH;
constexpr int OFF_PP = OFF_ND + 2 * CH;
constexpr int OFF_DSP = OFF_PP + 2 * CH;
constexpr int OFF_PADKV = OFF_DSP + 2 * CH;
constexpr int OFF_PADW = OFF_PADKV + 2 * D;
constexpr int LDS = OFF_PADW + THREADS;
constexpr int OFF_ROWS = 2 * BUF;      // finished rows: two tensors of TB rows (OFF_Y's buffers)
static_assert(2 * 4 * NW * 64 * 4 <= OFF_ROWS && OFF_ROWS + 2 * TB * D <= OFF_LH, "the merge fits in the row buffers");
static_assert(2 * LDS * 4 <= 160 * 1024, "two workgroups per compute unit");
static_assert(THREADS == 2 * kPadPartial, "two threads per pad-gradient channel");

// Row r holds its 16-byte piece p at position p ^ (r & 15): the 16 rows a 16-lane read of one
// piece touches cover all 64 banks.
__device__ __forceinline__ int swz(int r) { return r & 15; }

// the second part of LSE log2(e), lh = LSE kLog2eHi being the first (0 where that is infinite: a
// query whose LSE the caller sets to +inf has P = 0)
__device__ __forceinline__ float lse_low(float lse, float lh) {
    const float ll = __builtin_fmaf(lse, kLog2eLo, __builtin_fmaf(lse, kLog2eHi, -lh));
    return __builtin_fabsf(lh) < INFINITY ? ll : 0.f;
}
__device__ __forceinline__ float dot4(const float4& x, const float4& y, float s) {
    s = __builtin_fmaf(x.x, y.x, s);
    s = __builtin_fmaf(x.y, y.y, s);
    s = __builtin_fmaf(x.z, y.z, s);
    return __builtin_fmaf(x.w, y.w, s);
}
__device__ __forceinline__ float4 load4(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(float4, bload16(r, off));
}
__device__ __forceinline__ float4 lds4(const float* p) { return *reinterpret_cast<const float4*>(p); }

// What both roles know about their block, and the lane's operand addresses in a chunk's rows.
struct Block {
    int b, win, blk, head;
    WindowRect wr;
    int n;                      // tokens of the window
    long long n_pad;            // virtual key slots of its canvas square (KV-token mode)
    WindowAddr addr;
    long long q_base, kv_base, pad_elems;   // elements to the window's first token, and to the pad row
    __amdgpu_buffer_rsrc_t qr, orr, dor, kr, vr, lr;
    int tid, lane, li, h, wave, tt, sh;
    int rb;                     // row read: piece h D/8 + j of row 32 sh + li at rb ^ 4 j
    int cb[4];                  // column read of row 32 sh + 8 q + 4 h + j: see column()
};

// element 32 db + li of row 32 sh + 8 (r / 4) + 4 h + r % 4 of a chunk's rows
__device__ __forceinline__ float column(const Block& k, const float* rows, int r, int db) {
    const int q = r >> 2;
    return rows[k.cb[r & 3] + 8 * q * D + 32 * (db ^ (q & 1))];
}

// the lane's half of 32 row-read channels: acc += <streamed row, reg> over them
__device__ __forceinline__ floatx16 row_product(const Block& k, const float* rows, const float (&reg)[D / 2],
                                                floatx16 acc) {
#pragma unroll
    for (int j = 0; j < D / 8; ++j) {
        const float4 x = lds4(rows + (k.rb ^ (4 * j)));
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.x, reg[4 * j], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.y, reg[4 * j + 1], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.z, reg[4 * j + 2], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.w, reg[4 * j + 3], acc, 0, 0, 0);
    }
    return acc;
}

// Rows 16 w .. 16 w + 15 of the chunk starting at window-local token `base` straight into the
// swizzled LDS rows `dst`; rows past the window: zeros (LAST: the window's last row).
template <bool LAST = false>
__device__ __forceinline__ void load_rows(const Block& k, __amdgpu_buffer_rsrc_t src, float* dst, int base) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 16 * k.wave + 4 * i + (k.lane >> 4);
        const int p = (k.lane & 15) ^ swz(r);
        const int t = base + r;
        const unsigned off = LAST ? k.addr(min(t, k.n - 1)) + 16 * p : t < k.n ? k.addr(t) + 16 * p : kOutside;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(src, (lds_void*)(dst + (16 * k.wave + 4 * i) * D), 16, off, 0, 0, 0);
    }
}

// the lane's half (channels h D/2 ..) of a token's row, times `scale`
__device__ __forceinline__ void load_half(const Block& k, __amdgpu_buffer_rsrc_t src, int t, float (&reg)[D / 2],
                                          float scale) {
    const unsigned off = t < k.n ? k.addr(t) + k.h * (D / 2) * 4 : kOutside;
#pragma unroll
    for (int i = 0; i < D / 8; ++i) {
        const float4 x = load4(src, off + 16 * i);
        reg[4 * i] = x.x * scale;
        reg[4 * i + 1] = x.y * scale;
        reg[4 * i + 2] = x.z * scale;
        reg[4 * i + 3] = x.w * scale;
    }
}

// The two waves of a tile add their accumulators: each hands over the row groups that its
// partner finishes (of every channel block 2 sh', 2 sh' + 1) ...
__device__ __forceinline__ void hand_over(const Block& k, float4* exch, const floatx16 (&acc)[2]) {
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int lo = 4 * i, hi = 8 + 4 * i;
            exch[((k.wave * 2 + db) * 2 + i) * 64 + k.lane] =
                k.sh ? make_float4(acc[db][lo], acc[db][lo + 1], acc[db][lo + 2], acc[db][lo + 3])
                     : make_float4(acc[db][hi], acc[db][hi + 1], acc[db][hi + 2], acc[db][hi + 3]);
        }
}
// ... and finishes its own: (sum + w[ch] extra) * scale into the tile's staged rows.  The sum is wave
// sh = 0's part plus wave sh = 1's in both.
__device__ __forceinline__ void finish(const Block& k, const float4* exch, float* rows, const floatx16 (&acc)[2],
                                       float scale, float extra, const float* w) {
    const int row = TL * k.tt + k.li;
#pragma unroll
    for (int db = 0; db < 2; ++db)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int lo = 4 * i, hi = 8 + 4 * i, ch = 32 * db + 8 * (2 * k.sh + i) + 4 * k.h;
            const float4 y = exch[(((k.wave ^ 1) * 2 + db) * 2 + i) * 64 + k.lane];
            float4 x = k.sh ? make_float4(acc[db][hi], acc[db][hi + 1], acc[db][hi + 2], acc[db][hi + 3])
                            : make_float4(acc[db][lo], acc[db][lo + 1], acc[db][lo + 2], acc[db][lo + 3]);
            x = make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
            if (w != nullptr) {
                const float4 e = lds4(w + ch);
                x = make_float4(__builtin_fmaf(extra, e.x, x.x), __builtin_fmaf(extra, e.y, x.y),
                                __builtin_fmaf(extra, e.z, x.z), __builtin_fmaf(extra, e.w, x.w));
            }
            *reinterpret_cast<float4*>(rows + row * D + 4 * ((ch >> 2) ^ swz(row))) =
                make_float4(x.x * scale, x.y * scale, x.z * scale, x.w * scale);
        }
}
// the block's staged rows to their tokens, whole 256-byte rows
__device__ __forceinline__ void store_rows(const Block& k, const float* rows, __amdgpu_buffer_rsrc_t dst) {
#pragma unroll
    for (int i = k.tid; i < TB * ROWP; i += THREADS) {
        const int r = i / ROWP, p = i % ROWP, t = TB * k.blk + r;
        const u32x4 v = *reinterpret_cast<const u32x4*>(rows + r * D + 4 * (p ^ swz(r)));
        __builtin_amdgcn_raw_buffer_store_b128(v, dst, t < k.n ? k.addr(t) + 16 * p : kOutside, 0, 0);
    }
}

template <bool KVPAD>
__device__ __forceinline__ void key_role(const SwinBwdArgs& ba, const Block& k, float* smem) {
    const SwinArgs& a = ba.f;
    const int key0 = TB * k.blk;
    if (key0 >= k.n) return;   // the window has fewer blocks
    const bool pad_here = KVPAD && k.n_pad > 0 && k.blk == 0;
    if (KVPAD && k.blk == 0 && !pad_here && k.tid < kPadPartial) {   // the reduction reads a dense array
        const long long e = ((long long)k.b * a.heads + k.head) * a.n_windows + k.win;
        ba.ws[e * kPadPartial + k.tid] = 0.f;
    }
    const bool work = key0 + TL * k.tt < k.n;
    const int nch = (k.n + CH - 1) / CH;
    float* padkv = smem + OFF_PADKV;

    // the row this thread prepares of every chunk (4 threads per row: pieces qq, qq + 4, ...)
    const int pr = 16 * k.wave + (k.lane >> 2), qq = k.lane & 3;
    float4 ov[4];
    float lse;
    auto issue = [&](int c) {
        const int buf = c & 1, t = CH * c + pr;
        load_rows<true>(k, k.qr, smem + OFF_X + buf * BUF, CH * c);
        load_rows(k, k.dor, smem + OFF_Y + buf * BUF, CH * c);
        const unsigned off = t < k.n ? k.addr(t) + 16 * qq : kOutside;
#pragma unroll
        for (int i = 0; i < 4; ++i) ov[i] = load4(k.orr, off + 64 * i);
        lse = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(
                                            k.lr, t < k.n ? 4 * k.addr.token(t, (unsigned)k.wr.W) : kOutside, 0, 0));
    };
    issue(0);
    float kreg[D / 2], vreg[D / 2];
    load_half(k, k.kr, key0 + TL * k.tt + k.li, kreg, a.scale_log2);
    load_half(k, k.vr, key0 + TL * k.tt + k.li, vreg, 1.f);
    if (pad_here) {
        if (k.tid < 2 * D)
            padkv[k.tid] = static_cast<const float*>(k.tid < D ? a.k : a.v)[k.pad_elems + (k.tid & (D - 1))];
        __syncthreads();
    }
    const float log2_npad = pad_here ? log2f((float)k.n_pad) : 0.f;
    float pad_sum = 0.f;   // thread (half, channel): its half of each chunk's rows, over the chunks

    floatx16 dkT[2] = {floatx16{}, floatx16{}}, dvT[2] = {floatx16{}, floatx16{}};
    for (int c = 0; c < nch; ++c) {
        const int buf = c & 1;
        float* Qs = smem + OFF_X + buf * BUF;
        float* Gs = smem + OFF_Y + buf * BUF;
        float* LH = smem + OFF_LH + buf * CH;
        float* LL = smem + OFF_LL + buf * CH;
        float* ND = smem + OFF_ND + buf * CH;
        float* PP = smem + OFF_PP + buf * CH;
        float* DSP = smem + OFF_DSP + buf * CH;
        // ---- the wave's own rows of this chunk: LSE log2(e), D and the pad token's P and dS.  Rows past
        // the window get an LSE of +inf, which makes P zero: their Q is that of the window's last row, since
        // the logit of a zero row and a key with an infinite component would be 0 * inf
        wait_loads();
        {
            float dd = 0.f, zp = 0.f, dp = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int p = qq + 4 * i, at = pr * D + 4 * (p ^ swz(pr));
                const float4 g4 = lds4(Gs + at);
                dd = dot4(g4, ov[i], dd);
                if (pad_here) {
                    zp = dot4(lds4(Qs + at), lds4(padkv + 4 * p), zp);
                    dp = dot4(g4, lds4(padkv + D + 4 * p), dp);
                }
            }
            dd += __shfl_xor(dd, 1);
            dd += __shfl_xor(dd, 2);
            if (CH * c + pr >= k.n) lse = INFINITY;
            const float lh = lse * kLog2eHi;
            const float ll = lse_low(lse, lh);
            if (pad_here) {
                zp += __shfl_xor(zp, 1);
                zp += __shfl_xor(zp, 2);
                dp += __shfl_xor(dp, 1);
                dp += __shfl_xor(dp, 2);
                const float p = CH * c + pr < k.n ? exp2f(__builtin_fmaf(zp, a.scale_log2, log2_npad - lh) - ll) : 0.f;
                if (qq == 0) {
                    PP[pr] = p;
                    DSP[pr] = p * (dp - dd);
                }
            }
            if (qq == 0) {
                LH[pr] = lh;
                LL[pr] = ll;
                ND[pr] = -dd;
            }
        }
        __syncthreads();   // the chunk is published; every wave is done with the previous one
        if (c + 1 < nch) issue(c + 1);
        if (pad_here) {
            // thread (half, ch) sums channel ch of dS_p q (ch < 64) or P_p dO over rows 32 half ..
            // + 31 (rows past the window have P = dS = 0)
            const int ch = k.tid & (D - 1), half = k.tid / kPadPartial;
            const bool is_k = (k.tid & (kPadPartial - 1)) < D;
            const float* w = is_k ? DSP : PP;
            const float* rows = is_k ? Qs : Gs;
            float s4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int i = 0; i < CH / 2; i += 4)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int r = CH / 2 * half + i + j;
                    s4[j] = __builtin_fmaf(w[r], rows[r * D + 4 * ((ch >> 2) ^ swz(r)) + (ch & 3)], s4[j]);
                }
            pad_sum += (s4[0] + s4[1]) + (s4[2] + s4[3]);
        }
        if (!work || CH * c + TL * k.sh >= k.n) continue;
        // ---- the streamed tile (register r: query 8 (r / 4) + 4 h + r % 4) against the wave's keys
        const floatx16 s = row_product(k, Qs, kreg, floatx16{});
        floatx16 dp;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 d4 = lds4(ND + TL * k.sh + 8 * i + 4 * k.h);
            dp[4 * i] = d4.x;
            dp[4 * i + 1] = d4.y;
            dp[4 * i + 2] = d4.z;
            dp[4 * i + 3] = d4.w;
        }
        dp = row_product(k, Gs, vreg, dp);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 h4 = lds4(LH + TL * k.sh + 8 * i + 4 * k.h), l4 = lds4(LL + TL * k.sh + 8 * i + 4 * k.h);
            const float hv[4] = {h4.x, h4.y, h4.z, h4.w}, lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int r = 4 * i + j;
                const float p = __builtin_amdgcn_exp2f((s[r] - hv[j]) - lv[j]);
                const float ds = p * dp[r];
#pragma unroll
                for (int db = 0; db < 2; ++db) {
                    dvT[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(column(k, Gs, r, db), p, dvT[db], 0, 0, 0);
                    dkT[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(column(k, Qs, r, db), ds, dkT[db], 0, 0, 0);
                }
            }
        }
    }
    if (pad_here) smem[OFF_PADW + k.tid] = pad_sum;
    __syncthreads();   // the row buffers are free; the pad sums are complete
    if (pad_here && k.tid < kPadPartial) {
        const long long e = ((long long)k.b * a.heads + k.head) * a.n_windows + k.win;
        const float x = smem[OFF_PADW + k.tid] + smem[OFF_PADW + kPadPartial + k.tid];
        ba.ws[e * kPadPartial + k.tid] = k.tid < D ? x * ba.scale : x;
    }
    float4* exch_k = reinterpret_cast<float4*>(smem);
    float4* exch_v = exch_k + NW * 4 * 64;
    float* rows_k = smem + OFF_ROWS;
    float* rows_v = rows_k + TB * D;
    if (work) {
        hand_over(k, exch_k, dkT);
        hand_over(k, exch_v, dvT);
    }
    __syncthreads();
    if (work) {
        finish(k, exch_k, rows_k, dkT, ba.scale, 0.f, nullptr);
        finish(k, exch_v, rows_v, dvT, 1.f, 0.f, nullptr);
    }
    __syncthreads();
    const long long kv_bytes = ((long long)a.B * a.kv_batch_stride - k.kv_base) * 4;
    store_rows(k, rows_k, make_rsrc(static_cast<float*>(ba.dk) + k.kv_base, kv_bytes));
    store_rows(k, rows_v, make_rsrc(static_cast<float*>(ba.dv) + k.kv_base, kv_bytes));
}

template <bool KVPAD>
__device__ __forceinline__ void query_role(const SwinBwdArgs& ba, const Block& k, float* smem) {
    const SwinArgs& a = ba.f;
    const int q0 = TB * k.blk;
    if (q0 >= k.n) return;
    const bool has_pad = KVPAD && k.n_pad > 0;
    const int q = q0 + TL * k.tt + k.li;   // the lane's query
    const bool work = q0 + TL * k.tt < k.n;
    const int nch = (k.n + CH - 1) / CH;
    float* padkv = smem + OFF_PADKV;
    auto issue = [&](int c) {
        load_rows(k, k.kr, smem + OFF_X + (c & 1) * BUF, CH * c);
        load_rows(k, k.vr, smem + OFF_Y + (c & 1) * BUF, CH * c);
    };
    issue(0);
    float qreg[D / 2], greg[D / 2];
    load_half(k, k.qr, q, qreg, a.scale_log2);
    load_half(k, k.dor, q, greg, 1.f);
    float dd = 0.f;
    {
        const unsigned off = q < k.n ? k.addr(q) + k.h * (D / 2) * 4 : kOutside;
#pragma unroll
        for (int i = 0; i < D / 8; ++i)
            dd = dot4(make_float4(greg[4 * i], greg[4 * i + 1], greg[4 * i + 2], greg[4 * i + 3]),
                      load4(k.orr, off + 16 * i), dd);
    }
    dd = xhalf_sum(dd);
    const float lse = __builtin_bit_cast(
        float, __builtin_amdgcn_raw_buffer_load_b32(k.lr, q < k.n ? 4 * k.addr.token(q, (unsigned)k.wr.W) : kOutside, 0, 0));
    const float lh = lse * kLog2eHi;
    const float ll = lse_low(lse, lh);
    // pad token as key: dS_p = n_pad exp(c <q, k_pad> - LSE) (<dO, v_pad> - D); dq gets dS_p k_pad
    float dsp = 0.f;
    if (has_pad) {
        if (k.tid < 2 * D)
            padkv[k.tid] = static_cast<const float*>(k.tid < D ? a.k : a.v)[k.pad_elems + (k.tid & (D - 1))];
        __syncthreads();
        float zp = 0.f, dp = 0.f;
#pragma unroll
        for (int i = 0; i < D / 2; ++i) {
            zp = __builtin_fmaf(qreg[i], padkv[k.h * (D / 2) + i], zp);
            dp = __builtin_fmaf(greg[i], padkv[D + k.h * (D / 2) + i], dp);
        }
        zp = xhalf_sum(zp);
        dp = xhalf_sum(dp);
        dsp = exp2f((zp + (log2f((float)k.n_pad) - lh)) - ll) * (dp - dd);
    }

    floatx16 dqT[2] = {floatx16{}, floatx16{}};
    for (int c = 0; c < nch; ++c) {
        const float* Ks = smem + OFF_X + (c & 1) * BUF;
        const float* Vs = smem + OFF_Y + (c & 1) * BUF;
        wait_loads();
        __syncthreads();   // the chunk is published; every wave is done with the previous one
        if (c + 1 < nch) issue(c + 1);
        const int nv = k.n - (CH * c + TL * k.sh);   // keys of the wave's tile
        if (!work || nv <= 0) continue;
        floatx16 s = row_product(k, Ks, qreg, floatx16{});
        floatx16 dp;
#pragma unroll
        for (int r = 0; r < 16; ++r) dp[r] = -dd;
        dp = row_product(k, Vs, greg, dp);
        // register r: key 8 (r / 4) + 4 h + r % 4; rows past the window are zero, and P is cleared so
        // that no infinity meets them
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float p = __builtin_amdgcn_exp2f((s[r] - lh) - ll);
            s[r] = (8 * (r >> 2) + 4 * k.h + (r & 3) < nv ? p : 0.f) * dp[r];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int db = 0; db < 2; ++db)
                dqT[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(column(k, Ks, r, db), s[r], dqT[db], 0, 0, 0);
    }
    __syncthreads();   // the row buffers are free
    float4* exch = reinterpret_cast<float4*>(smem);
    float* rows = smem + OFF_ROWS;
    if (work) hand_over(k, exch, dqT);
    __syncthreads();
    if (work) finish(k, exch, rows, dqT, ba.scale, dsp, has_pad ? padkv : nullptr);
    __syncthreads();
    store_rows(k, rows, make_rsrc(static_cast<float*>(ba.dq) + k.q_base, ((long long)a.B * a.q_batch_stride - k.q_base) * 4));
}

// Workgroup id -> (unit, block, role), unit = (batch entry, window, head): the workgroups of one
// unit get ids that are equal mod 8, one after the other, so that they run on one XCD and all but
// the first find the window's rows in its L2.
template <bool KVPAD>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
void swin_bwd_f32_kernel(SwinBwdArgs ba) {
    const SwinArgs& a = ba.f;
    __shared__ __attribute__((aligned(16))) float smem[LDS];
    const unsigned id = blockIdx.x + kGridX * blockIdx.y;
    const unsigned rest = id >> 3;
    const unsigned g = ba.div_2nbb.div(rest);
    const unsigned j = rest - g * (2u * (unsigned)ba.nbb);
    const unsigned unit = (g << 3) + (id & 7u);
    if (unit >= (unsigned)a.n_units) return;
    Block k;
    k.blk = (int)(j >> 1);
    const unsigned i2 = a.div_heads.div(unit);
    k.head = (int)(unit - i2 * (unsigned)a.heads);
    const unsigned i3 = a.div_nwin.div(i2);
    k.win = (int)(i2 - i3 * (unsigned)a.n_windows);
    k.b = (int)i3;
    k.wr = window_rect<true>(a, k.win);
    k.n = k.wr.rows * k.wr.cols;
    k.n_pad = (long long)a.window * a.window - k.n;

    const long long win_elems = k.wr.tok0 * a.tok_stride + k.head * D;
    k.q_base = (long long)k.b * a.q_batch_stride + win_elems;
    k.kv_base = (long long)k.b * a.kv_batch_stride + win_elems;
    k.pad_elems = (long long)k.b * a.kv_batch_stride + a.L * a.tok_stride + k.head * D;
    const long long q_bytes = ((long long)a.B * a.q_batch_stride - k.q_base) * 4;
    const long long kv_bytes = ((long long)a.B * a.kv_batch_stride - k.kv_base) * 4;
    k.qr = make_rsrc(static_cast<const float*>(a.q) + k.q_base, q_bytes);
    k.orr = make_rsrc(static_cast<const float*>(ba.out) + k.q_base, q_bytes);
    k.dor = make_rsrc(static_cast<const float*>(ba.dout) + k.q_base, q_bytes);
    k.kr = make_rsrc(static_cast<const float*>(a.k) + k.kv_base, kv_bytes);
    k.vr = make_rsrc(static_cast<const float*>(a.v) + k.kv_base, kv_bytes);
    const long long lse_base = ((long long)k.b * a.heads + k.head) * a.L + k.wr.tok0;
    const long long lse_total = (long long)a.B * a.heads * a.L;
    k.lr = make_rsrc(ba.lse + lse_base, (lse_total - lse_base) * 4);
    k.addr.init(k.wr.cols, (unsigned)((long long)k.wr.W * a.tok_stride * 4), (unsigned)(a.tok_stride * 4));

    k.tid = (int)threadIdx.x;
    k.lane = k.tid & 63;
    k.li = k.lane & 31;
    k.h = k.lane >> 5;
    k.wave = __builtin_amdgcn_readfirstlane(k.tid >> 6);
    k.tt = k.wave >> 1;
    k.sh = k.wave & 1;
    k.rb = (TL * k.sh + k.li) * D + 4 * ((k.h * (D / 8)) ^ swz(k.li));
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int row = 4 * k.h + c;
        k.cb[c] = (TL * k.sh + row) * D + 4 * ((k.li >> 2) ^ swz(row)) + (k.li & 3);
    }
    if (j & 1u)
        query_role<KVPAD>(ba, k, smem);
    else
        key_role<KVPAD>(ba, k, smem);
}

// One workgroup per (batch entry, head): row L of dk and dv = the sum of the partials of
// every (window, query block).  1024 threads = 8 slices x 128 columns; slice s adds entries
// s, s + 8, ... in their order, fetching 32 of them at a time (one memory round trip per 32
// instead of one per few), and the eight slice sums are added in order.
constexpr int kRedSlices = 8;
constexpr int kRedBatch = 32;
template <typename T>
__global__ __launch_bounds__(kRedSlices * kPadPartial) void swin_bwd_pad_reduce_kernel(SwinBwdArgs ba) {
    const SwinArgs& a = ba.f;
    __shared__ float part[kRedSlices][kPadPartial];
    const int bh = blockIdx.x;
    const int col = threadIdx.x % kPadPartial;
    const int slice = threadIdx.x / kPadPartial;
    const long long nent = (long long)a.n_windows * ba.pad_blocks;
    const float* src = ba.ws + (long long)bh * nent * kPadPartial + col;
    float acc = 0.f;
    for (long long e0 = slice; e0 < nent; e0 += (long long)kRedBatch * kRedSlices) {
        float v[kRedBatch];
#pragma unroll
        for (int u = 0; u < kRedBatch; ++u) {
            const long long e = e0 + (long long)u * kRedSlices;
            v[u] = e < nent ? src[e * kPadPartial] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < kRedBatch; ++u) acc += v[u];
    }
    part[slice][col] = acc;
    __syncthreads();
    if (slice == 0) {
        float s = part[0][col];
        for (int i = 1; i < kRedSlices; ++i) s += part[i][col];
        const int b = bh / a.heads, head = bh - b * a.heads;
        const long long row = (long long)b * a.kv_batch_stride + a.L * a.tok_stride + head * D;
        T* dst = static_cast<T*>(col < D ? ba.dk : ba.dv) + row + (col % D);
        if constexpr (sizeof(T) == 2) {
            const __bf16 r = (__bf16)s;
            *dst = __builtin_bit_cast(uint16_t, r);
        } else {
            *dst = s;
        }
    }
}

}  // namespace

hipError_t launch_swin_bwd_f32(const SwinBwdArgs& a, hipStream_t stream) {
    SwinBwdArgs args = a;
    args.nbb = (a.f.n_max + TB - 1) / TB;
    args.div_2nbb = FastDiv::make(2u * (unsigned)args.nbb);
    void* params[] = {&args};
    const void* fn = a.f.pad_mode == 1 ? reinterpret_cast<const void*>(&swin_bwd_f32_kernel<true>)
                                       : reinterpret_cast<const void*>(&swin_bwd_f32_kernel<false>);
    // up to eight times as many workgroups as the host's limit counts (blocks of 256 tokens): ids
    // past one row of the launch grid go on along y
    const int64_t groups = 16 * (int64_t)args.nbb * ((a.f.n_units + 7) / 8);
    const unsigned gy = (unsigned)((groups + kGridX - 1) / kGridX);
    return hipLaunchKernel(fn, dim3(gy > 1 ? kGridX : (unsigned)groups, gy), dim3(THREADS), params, 0, stream);
}

hipError_t launch_swin_bwd_pad_reduce(const SwinBwdArgs& a, int elem_bytes, hipStream_t stream) {
    SwinBwdArgs args = a;
    void* params[] = {&args};
    const void* fn = elem_bytes == 2 ? reinterpret_cast<const void*>(&swin_bwd_pad_reduce_kernel<uint16_t>)
                                     : reinterpret_cast<const void*>(&swin_bwd_pad_reduce_kernel<float>);
    return hipLaunchKernel(fn, dim3((unsigned)(a.f.B * a.f.heads)), dim3(kRedSlices * kPadPartial), params, 0,
                           stream);
}

}  // namespace fla

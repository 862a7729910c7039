// Flash Swin attention forward, fp32 storage and arithmetic, gfx950 (CDNA4) matrix cores.
//
// One workgroup = one (batch entry, window, block of 64 queries, head), 256 threads = 4
// waves: wave (qt, kh) takes the 32 queries of tile qt of the block against every other
// 32-key tile of the window (tiles kh, kh + 2, ...); the two waves of a query tile merge
// their softmax states at the end.
//
// Products run on v_mfma_f32_32x32x2_f32 (fp32 operands, fp32 accumulation):
//   S^T = K . Q^T   lane (i, h) = (l % 32, l / 32) supplies channel h D/2 + s of key row i (A,
//                   from LDS, 16 bytes at a time) and of query i (B, in registers) at step
//                   s: the order of the channels in the sum is free as long as both operands
//                   agree.  The lane then holds the 16 keys 8 (r / 4) + 4 h + r % 4 of query i.
//   O^T += V^T . P^T   step r sums keys key(r, 0) and key(r, 1): the lane's B operand is its
//                   own p[r], with no exchange between lanes, and its A operand is
//                   V[key(r, h)][channel], a row-major read.
//
// Keys stream through LDS 64 at a time (two tiles, one per kh) by buffer loads that write
// LDS, into one buffer: while one workgroup waits for its rows, the two others of the compute
// unit (34 KB of LDS and at most 168 VGPRs each) keep the matrix cores busy.  The 16-byte
// pieces of a row are XOR-swizzled by the row, which spreads the 16-byte row reads over the
// banks.
//
// Bound by the fp32 matrix rate (64 flop per cycle and SIMD, 157 TFLOP/s): a 32 x 32 tile is
// 64 products of 64 cycles at D = 64, beside ~170 vector and ~40 LDS instructions that the
// other waves of the SIMD hide.
// Measured, 12 heads of 64: 128x128 tokens, window 32: 425 us (121 TFLOP/s); 64x64 tokens, window
// 16, shift 8: 40 us.  One query per thread on the vector ALU with the keys broadcast from LDS
// (bound by those broadcasts, one wave per SIMD) took 2250 and 290 us.  64 queries and two waves
// per query tile keep the pieces small, since a 64x64 grid has 300 (window, head) units of
// unequal size for 256 compute units: blocks of 128 queries with double-buffered rows took 42 us
// there and 141 against 113 us at window 64, for 409 us at 128x128.
//
// KV-only padding (Sec. 3.4, App. B): the pad token is key n with logit + log2(n_pad).
// RoPE (Sec. 3.1): q and k are rotated with angles, sine and cosine in double, k in place in
// LDS, from a table of the window's row and column positions where its rectangle fits
// 32 x 32 and per 4 channels otherwise (the same expression: the same bits).
#include "fla_swin_device.h"

namespace fla {
namespace {

constexpr int THREADS = 256;
constexpr int NW = THREADS / 64;
constexpr int TL = 32;                 // queries (keys) per tile
constexpr int QB = 2 * TL;             // queries per workgroup: two waves per tile
constexpr int KC = 2 * TL;             // keys per LDS chunk: one tile per kh
constexpr int kRopeTab = 32;           // window rows / columns covered by the RoPE table

constexpr float kLn2Hi = 0.693147182f, kLn2Lo = -1.90465430e-9f;

template <int D>
struct Cfg {
    static constexpr int ROWP = D / 4;          // 16-byte pieces per row
    static constexpr int NB = D / 32;           // channel blocks of O^T
    static constexpr int BUF = KC * D;          // floats of the K (V) rows in LDS
    static constexpr int OS = D + 4;            // stride of the staged output rows, floats
    // after the last chunk LDS holds the exchanged halves of O^T, the merged rows and (m, l)
    static constexpr int OFF_ROWS = NW * NB * 2 * 64 * 4;
    static constexpr int OFF_ML = OFF_ROWS + QB * OS;
    static constexpr int LDS = OFF_ML + NW * TL * 2;
    static_assert(LDS >= 2 * BUF, "K and V rows");
    // q and o take D floats per lane: 2 waves per SIMD at D = 128, and 3 at D = 64, where 4 spill
    // (43.6 against 40 us at 64x64 tokens)
    static constexpr int WAVES = D > 64 ? 2 : 3;
};

// Row r of a chunk holds its 16-byte piece p at position p ^ swz(r), so that the 16 rows a
// 16-lane read of one piece touches cover all 64 banks (at D = 32 two rows share them).
template <int D>
__device__ __forceinline__ int swz(int r) {
    return D == 32 ? (r >> 1) & 7 : r & 15;
}

template <int D, bool ROPE>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(ROPE ? 2 : Cfg<D>::WAVES, ROPE ? 2 : Cfg<D>::WAVES)))
void swin_fwd_f32_kernel(SwinArgs a) {
    using C = Cfg<D>;
    constexpr int ROWP = C::ROWP, NB = C::NB;
    __shared__ __attribute__((aligned(16))) float smem[C::LDS];
    __shared__ double Rtab[ROPE ? 2 * kRopeTab * (D / 4) * 2 : 1];    // [axis][position][frequency] (cos, sin)
    float* Ks = smem;
    float* Vs = smem + C::BUF;

    // ---- workgroup -> (unit, query block): the blocks of one unit (b, window, head) on one
    //      XCD, one after the other, so that all but the first reader of its K and V find them in L2
    const unsigned id = blockIdx.x + kGridX * blockIdx.y;
    const unsigned rest = id >> 3;
    const unsigned g = a.div_nqb.div(rest);
    const int qblk = (int)(rest - g * (unsigned)a.nqb);
    const unsigned unit = (g << 3) + ((id + (g >> 2)) & 7u);
    if (unit >= (unsigned)a.n_units) return;
    const unsigned id2 = a.div_heads.div(unit);
    const int head = (int)(unit - id2 * (unsigned)a.heads);
    const unsigned id3 = a.div_nwin.div(id2);
    const int win = (int)(id2 - id3 * (unsigned)a.n_windows);
    const int b = (int)id3;

    const WindowRect wr = window_rect<true>(a, win);
    const int n = wr.rows * wr.cols;
    const int q_begin = qblk * QB;
    if (q_begin >= n) return;

    const long long n_pad = (long long)a.window * a.window - n;
    const bool has_pad = a.pad_mode == 1 && n_pad > 0;
    const int nk = n + (has_pad ? 1 : 0);
    const float pad_bias = has_pad ? log2f((float)n_pad) : 0.f;

    const long long win_elems = wr.tok0 * a.tok_stride + head * D;
    const long long q_base = (long long)b * a.q_batch_stride + win_elems;
    const long long kv_base = (long long)b * a.kv_batch_stride + win_elems;
    const long long q_bytes = ((long long)a.B * a.q_batch_stride - q_base) * 4;
    const long long kv_bytes = ((long long)a.B * a.kv_batch_stride - kv_base) * 4;
    const __amdgpu_buffer_rsrc_t qr = make_rsrc(static_cast<const float*>(a.q) + q_base, q_bytes);
    const __amdgpu_buffer_rsrc_t orr = make_rsrc(static_cast<float*>(a.out) + q_base, q_bytes);
    const __amdgpu_buffer_rsrc_t kr = make_rsrc(static_cast<const float*>(a.k) + kv_base, kv_bytes);
    const __amdgpu_buffer_rsrc_t vr = make_rsrc(static_cast<const float*>(a.v) + kv_base, kv_bytes);
    WindowAddr addr;
    addr.init(wr.cols, (unsigned)((long long)wr.W * a.tok_stride * 4), (unsigned)(a.tok_stride * 4));

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qt = wave >> 1, kh = wave & 1;
    const int li = lane & 31, h = lane >> 5;
    const int wq0 = q_begin + TL * qt;
    const int nq = min(TL, n - wq0);   // queries of this wave (<= 0: the wave only stages)

    // ---- staging: rows KW wave .. of chunk c straight into the swizzled LDS rows; lane L of the
    //      i-th load writes piece L % ROWP of row i RPL + L / ROWP.  Rows past the window: zeros.
    constexpr int RPL = 64 / ROWP, KW = KC / NW, LOADS = KW / RPL;
    auto issue = [&](int c) {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int r = KW * wave + RPL * i + lane / ROWP;
            const int t = KC * c + r, p = (lane % ROWP) ^ swz<D>(r);
            const unsigned off = t < n ? addr(t) + 16 * p : kOutside;
            const int base = (KW * wave + RPL * i) * D;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(kr, (lds_void*)(Ks + base), 16, off, 0, 0, 0);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(vr, (lds_void*)(Vs + base), 16, off, 0, 0, 0);
        }
    };
    issue(0);

    const bool rope_tab = ROPE && wr.rows <= kRopeTab && wr.cols <= kRopeTab;
    auto angle = [&](int axis, int p, int j) {   // of position p of the window along an axis, frequency j
        return (double)((axis ? wr.x0 : wr.y0) + p) * (double)a.rope_scale * a.rope_freq[j];
    };
    // rotate the two pairs of 4 channels starting at channel c0 of window-local token t
    auto rope4 = [&](float4& x, int t, int c0) {
        const unsigned r = mulhi_u32((unsigned)t, addr.magic) + ((unsigned)t & addr.one_mask);
        const int axis = c0 < D / 2 ? 0 : 1;
        const int p = axis ? (int)((unsigned)t - r * addr.cols) : (int)r;
        const int j = (c0 % (D / 2)) / 2;
        double s0, c0s, s1, c1s;
        if (rope_tab) {
            const double* cs = Rtab + ((axis * kRopeTab + p) * (D / 4) + j) * 2;
            c0s = cs[0];
            s0 = cs[1];
            c1s = cs[2];
            s1 = cs[3];
        } else {
            sincos(angle(axis, p, j), &s0, &c0s);
            sincos(angle(axis, p, j + 1), &s1, &c1s);
        }
        x = make_float4((float)(x.x * c0s - x.y * s0), (float)(x.y * c0s + x.x * s0),
                        (float)(x.z * c1s - x.w * s1), (float)(x.w * c1s + x.z * s1));
    };
    if constexpr (ROPE) {
        for (int e = tid; rope_tab && e < 2 * kRopeTab * (D / 4); e += THREADS) {
            const int axis = e / (kRopeTab * (D / 4)), p = (e / (D / 4)) % kRopeTab, j = e % (D / 4);
            double s, c;
            sincos(angle(axis, p, j), &s, &c);
            Rtab[2 * e] = c;
            Rtab[2 * e + 1] = s;
        }
        __syncthreads();
    }
    // the rows this wave loaded, published to the workgroup
    auto publish = [&](int c) {
        wait_loads();
        if constexpr (ROPE)
#pragma unroll 1
            for (int i = 0; i < LOADS; ++i) {   // each lane rotates the pieces it loaded
                const int r = KW * wave + RPL * i + lane / ROWP, t = KC * c + r;
                float4* x = reinterpret_cast<float4*>(Ks + (KW * wave + RPL * i) * D + 4 * lane);
                if (t < n) rope4(*x, t, 4 * ((lane % ROWP) ^ swz<D>(r)));
            }
        __syncthreads();
        const int slot = n - KC * c;
        if (has_pad && slot >= 0 && slot < KC) {   // the pad token is key n: over its zero-filled row
            if (tid < 2 * ROWP) {
                const long long pad_elems = (long long)b * a.kv_batch_stride + a.L * a.tok_stride + head * D;
                const float* src = static_cast<const float*>(tid < ROWP ? a.k : a.v) + pad_elems;
                const int p = tid % ROWP;
                *reinterpret_cast<float4*>((tid < ROWP ? Ks : Vs) + slot * D + 4 * (p ^ swz<D>(slot))) =
                    *reinterpret_cast<const float4*>(src + 4 * p);
            }
            __syncthreads();
        }
    };

    // ---- the lane's half of query li's channels, scaled to the exp2 domain
    float qv[D / 2];
    {
        const int tq = min(wq0 + li, n - 1);
        const unsigned row = addr(tq) + h * (D / 2) * 4;
#pragma unroll
        for (int i = 0; i < D / 8; ++i) {
            float4 x = __builtin_bit_cast(float4, bload16(qr, row + 16 * i));
            if constexpr (ROPE) rope4(x, tq, h * (D / 2) + 4 * i);
            qv[4 * i] = x.x * a.scale_log2;
            qv[4 * i + 1] = x.y * a.scale_log2;
            qv[4 * i + 2] = x.z * a.scale_log2;
            qv[4 * i + 3] = x.w * a.scale_log2;
        }
    }

    // operand addresses in LDS.  K: piece h D/8 + j of row 32 kh + li sits at kb ^ 4 j.  V: channel
    // 32 db + li of row 32 kh + key(r, h), key = 8 (r / 4) + 4 h + r % 4; the swizzle of that row
    // is a lane part (per r % 4, at D = 32 per r % 8) and a constant.
    const int kb = (TL * kh + li) * D + 4 * ((h * (D / 8)) ^ swz<D>(li));
    constexpr int NV = D == 32 ? 8 : 4;
    int vb[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int row = 8 * (j >> 2) + 4 * h + (j & 3);
        vb[j] = (TL * kh + row) * D + 4 * ((li >> 2) ^ swz<D>(row)) + (li & 3);
    }
    auto v_elem = [&](int r, int db) {
        const int q = r >> 2;
        return D == 32 ? Vs[vb[r & 7] + 16 * (q >> 1) * D]
                       : Vs[vb[r & 3] + 8 * q * D + 32 * (db ^ (q & 1))];
    };

    floatx16 o[NB];
#pragma unroll
    for (int db = 0; db < NB; ++db) o[db] = floatx16{};
    float m_run = -INFINITY, l_run = 0.f;
    const int nch = (nk + KC - 1) / KC;
    for (int c = 0; c < nch; ++c) {
        publish(c);
        const int t0 = KC * c + TL * kh;
        if (nq > 0 && t0 < nk) {
            floatx16 s = {};
#pragma unroll
            for (int j = 0; j < D / 8; ++j) {
                const float4 k4 = *reinterpret_cast<const float4*>(Ks + (kb ^ (4 * j)));
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.x, qv[4 * j], s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.y, qv[4 * j + 1], s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.z, qv[4 * j + 2], s, 0, 0, 0);
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(k4.w, qv[4 * j + 3], s, 0, 0, 0);
            }
            if (t0 + TL > n) {   // keys past the window's last, or the pad token
                const int lim = nk - (t0 + 4 * h), pad = n - (t0 + 4 * h);
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int off = 8 * (r >> 2) + (r & 3);
                    const float x = off == pad ? s[r] + pad_bias : s[r];
                    s[r] = off < lim ? x : -INFINITY;
                }
            }
            float mx = s[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = __builtin_fmaxf(mx, s[r]);
            mx = xhalf_max(mx);
            if (__builtin_amdgcn_ballot_w64(mx > m_run)) {
                const float m_new = __builtin_fmaxf(m_run, mx);
                const float alpha = m_new == m_run ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
                m_run = m_new;
                l_run *= alpha;
#pragma unroll
                for (int db = 0; db < NB; ++db) o[db] *= alpha;
            }
            const float m_sub = m_run == -INFINITY ? 0.f : m_run;   // every logit so far -inf: p = 0
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                s[r] = __builtin_amdgcn_exp2f(s[r] - m_sub);
                l_run += s[r];
            }
#pragma unroll
            for (int r = 0; r < 16; ++r)
#pragma unroll
                for (int db = 0; db < NB; ++db)
                    o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(v_elem(r, db), s[r], o[db], 0, 0, 0);
        }
        __syncthreads();   // every wave is done with the chunk
        if (c + 1 < nch) issue(c + 1);
    }

    // ---- merge the two waves of a query tile: each hands over half of its O^T (of every
    //      channel block the row groups that its partner finishes: 2 kh, 2 kh + 1) and its
    //      (m, l); the finished rows go through LDS so that every store writes whole rows
    float4* exch = reinterpret_cast<float4*>(smem);
    float* rows = smem + C::OFF_ROWS;
    float* ml = smem + C::OFF_ML;
    l_run = xhalf_sum(l_run);
    if (nq > 0) {
#pragma unroll
        for (int db = 0; db < NB; ++db)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int lo = 4 * i, hi = 8 + 4 * i;   // row group i (kh = 0) or 2 + i (kh = 1)
                const float4 x = kh ? make_float4(o[db][lo], o[db][lo + 1], o[db][lo + 2], o[db][lo + 3])
                                    : make_float4(o[db][hi], o[db][hi + 1], o[db][hi + 2], o[db][hi + 3]);
                exch[((wave * NB + db) * 2 + i) * 64 + lane] = x;
            }
        if (h == 0) {
            ml[(wave * TL + li) * 2] = m_run;
            ml[(wave * TL + li) * 2 + 1] = l_run;
        }
    }
    __syncthreads();
    if (nq > 0) {
        const int other = wave ^ 1;
        const float m_o = ml[(other * TL + li) * 2], l_o = ml[(other * TL + li) * 2 + 1];
        const float m = __builtin_fmaxf(m_run, m_o);
        const float w_me = m_run == m ? 1.f : __builtin_amdgcn_exp2f(m_run - m);
        const float w_o = m_o == m ? 1.f : __builtin_amdgcn_exp2f(m_o - m);
        // summed as wave kh = 0 then kh = 1 in both waves: one denominator per query
        const float l = kh ? __builtin_fmaf(l_o, w_o, l_run * w_me) : __builtin_fmaf(l_run, w_me, l_o * w_o);
        if (a.lse != nullptr && kh == 0 && h == 0 && li < nq)
            // ln 2 in two parts: m ln 2 + ln l with one rounding at the size of the result
            a.lse[((long long)b * a.heads + head) * a.L + wr.tok0 + addr.token(wq0 + li, (unsigned)wr.W)] =
                __builtin_fmaf(m, kLn2Hi, __builtin_fmaf(m, kLn2Lo, logf(l)));
        const float inv = 1.f / l;
        float* row = rows + (TL * qt + li) * C::OS + 4 * h;
#pragma unroll
        for (int db = 0; db < NB; ++db)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int lo = 4 * i, hi = 8 + 4 * i;
                const float4 y = exch[((other * NB + db) * 2 + i) * 64 + lane];
                const float4 x = kh ? make_float4(o[db][hi], o[db][hi + 1], o[db][hi + 2], o[db][hi + 3])
                                    : make_float4(o[db][lo], o[db][lo + 1], o[db][lo + 2], o[db][lo + 3]);
                *reinterpret_cast<float4*>(row + 32 * db + 8 * (2 * kh + i)) =
                    make_float4(__builtin_fmaf(y.x, w_o, x.x * w_me) * inv, __builtin_fmaf(y.y, w_o, x.y * w_me) * inv,
                                __builtin_fmaf(y.z, w_o, x.z * w_me) * inv, __builtin_fmaf(y.w, w_o, x.w * w_me) * inv);
            }
    }
    __syncthreads();
    const int nrows = min(QB, n - q_begin);
#pragma unroll
    for (int i = tid; i < QB * ROWP; i += THREADS) {
        const int r = i / ROWP, part = i % ROWP;
        const u32x4 v = *reinterpret_cast<const u32x4*>(rows + r * C::OS + 4 * part);
        const unsigned off = r < nrows ? addr(q_begin + r) + 16 * part : kOutside;   // past the window: dropped
        __builtin_amdgcn_raw_buffer_store_b128(v, orr, off, 0, 0);
    }
}

}  // namespace

hipError_t launch_swin_fwd_f32(const SwinArgs& a, hipStream_t stream) {
    SwinArgs args = a;
    args.nqb = (a.n_max + QB - 1) / QB;
    args.div_nqb = FastDiv::make((unsigned)args.nqb);
    void* params[] = {&args};
    const void* fn = a.rope              ? reinterpret_cast<const void*>(&swin_fwd_f32_kernel<kHeadDim, true>)
                     : a.head_dim == 32  ? reinterpret_cast<const void*>(&swin_fwd_f32_kernel<32, false>)
                     : a.head_dim == 128 ? reinterpret_cast<const void*>(&swin_fwd_f32_kernel<128, false>)
                                         : reinterpret_cast<const void*>(&swin_fwd_f32_kernel<kHeadDim, false>);
    // up to four times as many workgroups as the host's limit counts (blocks of 256 queries): ids
    // past one row of the launch grid go on along y
    const int64_t groups = 8 * (int64_t)args.nqb * ((a.n_units + 7) / 8);
    const unsigned gy = (unsigned)((groups + kGridX - 1) / kGridX);
    return hipLaunchKernel(fn, dim3(gy > 1 ? kGridX : (unsigned)groups, gy), dim3(THREADS), params, 0, stream);
}

}  // namespace fla

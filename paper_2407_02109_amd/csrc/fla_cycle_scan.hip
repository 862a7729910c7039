// Cycle-scan (HRSAM Sec. 3.5), fp32, gfx950: the selective state-space scan of every
// channel over the token sequence laid out `repeats` times, the output summed over the copies.
//
// Per channel and state (diagonal A, zero-order hold of the SSM equations of Sec. 3.5):
//   h_t = Abar_t h_{t-1} + Bbar_t x_t,  y_t = sum_n C_t[n] h_t[n],
//   Abar_t = exp(Delta_t a),  Bbar_t = (exp(Delta_t a) - 1) / a * B_t.
// The copies are never laid out.  The scan is linear in its initial state, so the state at
// token t of copy k + 1 is h1_t + P_t S_k, with h1 the scan of one copy from zero, P_t the
// decay from the sequence start to t and S_k the state at the end of copy k
// (S_k = (1 + P_L + ... + P_L^{k-1}) S_1).  Summed over the r copies:
//   sum_k h_t^(k) = r h1_t + P_t G,   G = sum_{j=0}^{r-2} (r-1-j) P_L^j S_1,
// which is the scan of r x started from G instead of zero.  Over chunks of T tokens:
//   pass A  (cycle_scan_chunks): every chunk scanned from zero; its output y1_t = C_t . h1_t
//           goes to y, its end state and its sum of Delta to the workspace;
//   pass B  (cycle_scan_carries): per (batch entry, channel, state), the chunks' carries in
//           order: the state entering chunk c, H_{c-1}, the state S_1 after the sequence, and
//           E_c = r H_{c-1} + P(start -> chunk c) G, the state from which chunk c of the summed
//           scan starts;
//   pass C  (cycle_scan_outputs): within chunk c the summed scan's state is r h1_t + P_t E_c
//           (P_t: the decay from the chunk's start to t), so y_t = r y1_t +
//           sum_n C_t[n] exp(a_n cum_t) E_c[n], cum_t the sum of Delta from the chunk's start
//           to t; no recurrence, y overwritten in place.
// Two passes of exponentials over the data, where scanning the laid-out copies takes r.
//
// A workgroup takes 64 channels of one chunk, a lane one channel; its SPLIT waves share the N
// states (N / SPLIT each in a lane's registers) and add their shares of y through LDS, four tokens
// at a time.  x (pass C: y1) and Delta of a token are one coalesced 256-byte read per wave; B_t and
// C_t, the same for every channel, are wave-uniform reads into scalar registers.
// Bound by the vector ALU: per (token, channel, state) pass A issues six plain operations and an
// exponential, pass C three and an exponential.  Measured with the operands in registers, a plain
// operation on vector registers takes 2.6 to 3.5 cycles of a SIMD with four or more waves on it
// (8 with one), one with a scalar operand 4.4 to 5, an exponential 8.5: about 30 and 20.4 cycles,
// 510 us for 65536 tokens x 768 channels x 32 states.  One wave per group ran them at 434 + 289 us
// (vector ALU busy 79 and 73%: waits for the scalar rows and a tail of unequal waves), four waves
// in pass A and one in pass C at 400 + 264 us; 4096 tokens, 768 groups for 1024 SIMDs: 118 -> 74 us
// a call with eight waves.  Taking the products over (tokens or states) x channels from the matrix
// cores (4x4x1 outer products, 9.5 cycles for four) was no faster: 690 us a call.
#include "fla_cycle_scan.h"

#include <type_traits>

#include "fla_swin_device.h"

namespace fla {
namespace {

constexpr float kLog2e = 1.4426950408889634f;
constexpr int kBatch = 32;   // chunk values per load batch of the carry pass
constexpr int kTokens = 4;   // tokens whose x and Delta the scan passes load together

// The N entries of a row of B or C.  The row is the same for the whole wave and read-only
// for the kernel's life: read through the constant address space, so that it comes in by
// scalar loads into scalar registers.
typedef __attribute__((address_space(4))) const float const_float;
template <int N>
__device__ __forceinline__ void load_row(const float* p, float (&w)[N]) {
    const const_float* q = (const const_float*)p;
#pragma unroll
    for (int n = 0; n < N; ++n) w[n] = q[n];
}

// What a wave of a scan pass works on: states ns .. ns + N / SPLIT - 1 of 64 channels of one chunk.
// Rows of x, Delta and y are addressed by a buffer resource at the row's first channel of the 64,
// whose range check drops the lanes past the last channel.
template <int N, int SPLIT>
struct ScanWave {
    static constexpr int NW = N / SPLIT;                                  // states per lane
    static constexpr int PER = SPLIT < kTokens ? kTokens / SPLIT : 1;     // tokens of a group this wave stores
    static constexpr int PAIR = N <= 8 || SPLIT > 1 ? 2 : 1;               // tokens whose rows are read together
    int lane, wave, b, chunk, t0, t1, ns, ch0, live_ch;
    size_t rb;
    __device__ __forceinline__ explicit ScanWave(const CycleArgs& c) {
        const int cg = blockIdx.x % c.cgroups;
        const int rest = blockIdx.x / c.cgroups;
        chunk = rest % c.nch;
        b = rest / c.nch;
        lane = (int)threadIdx.x & 63;
        wave = SPLIT > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) : 0;
        ns = wave * NW;
        ch0 = cg * 64;
        live_ch = min(64, c.d - ch0);
        t0 = chunk * c.T;
        t1 = min(t0 + c.T, c.L);
        rb = (size_t)b * c.L;
    }
    __device__ __forceinline__ bool ok() const { return lane < live_ch; }
    __device__ __forceinline__ int channel() const { return ch0 + min(lane, live_ch - 1); }
    // the lane's channel of token t of a [B, L, d] tensor
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t row(const CycleArgs& c, const float* p, int t) const {
        return make_rsrc(p + (rb + t) * c.d + ch0, 4 * live_ch);
    }
    __device__ __forceinline__ float load(const CycleArgs& c, const float* p, int t) const {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(row(c, p, t), 4u * (unsigned)lane, 0, 0));
    }
    __device__ __forceinline__ void store(const CycleArgs& c, float* p, int t, float v) const {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), row(c, p, t), 4u * (unsigned)lane, 0, 0);
    }
};

// f over the groups of kTokens tokens of [t0, t1): f(group's first token, tokens of it that exist),
// the whole groups with a compile-time count
template <typename F>
__device__ __forceinline__ void for_groups(int t0, int t1, F&& f) {
    const int tfull = t0 + (t1 - t0) / kTokens * kTokens;
    for (int tg = t0; tg < tfull; tg += kTokens) f(tg, std::integral_constant<int, kTokens>{});
    if (tfull < t1) f(tfull, t1 - tfull);
}

// The waves' shares of y of a group of tokens, added in wave order: wave w gets its PER tokens from
// PER w on in acc[0 ..].  One barrier per call: `red` alternates between two buffers.
template <int SPLIT, int PER>
__device__ __forceinline__ void add_shares(float (*red)[kTokens][64], int wave, int lane, float (&acc)[kTokens]) {
    if constexpr (SPLIT > 1) {
#pragma unroll
        for (int j = 0; j < kTokens; ++j) red[wave][j][lane] = acc[j];
        __syncthreads();
        if (PER * wave < kTokens)
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                float s = red[0][PER * wave + j][lane];
#pragma unroll
                for (int w = 1; w < SPLIT; ++w) s += red[w][PER * wave + j][lane];
                acc[j] = s;
            }
    }
}

// EARLY (one wave per group): every token's y is stored at once instead of with its group's, which takes
// 76 registers instead of 96 at 16 states, six waves per SIMD instead of five.
template <int N, int SPLIT, bool EARLY>
__global__ __launch_bounds__(64 * SPLIT) __attribute__((amdgpu_waves_per_eu(1, SPLIT >= 4 ? 6 : 8)))
void cycle_scan_chunks(CycleArgs c) {
    static_assert(!EARLY || SPLIT == 1, "the shares of y are added first");
    using W = ScanWave<N, SPLIT>;
    constexpr int NW = W::NW, PER = W::PER, PAIR = W::PAIR;
    __shared__ float red[2][SPLIT][kTokens][64];
    const W w(c);
    // the state scaled by a, g = a h, takes one product less per step:
    // g <- dA g + (dA - 1) u b; the output C . h = sum_n (C[n] / a[n]) g[n]
    float a2[NW], ia[NW], g[NW];
    const float* ap = c.A + (size_t)w.channel() * N + w.ns;
#pragma unroll
    for (int n = 0; n < NW; ++n) {
        const float a = ap[n];
        a2[n] = a * kLog2e;
        ia[n] = 1.f / a;
        g[n] = 0.f;
    }
    float sd = 0.f;
    int buf = 0;
    for_groups(w.t0, w.t1, [&](int tg, auto live) {
        float u[kTokens], dl[kTokens], acc[kTokens];
#pragma unroll
        for (int j = 0; j < kTokens; ++j) {
            u[j] = dl[j] = acc[j] = 0.f;
            if (j < live) {
                u[j] = w.load(c, c.x, tg + j);
                dl[j] = w.load(c, c.delta, tg + j);
            }
        }
#pragma unroll
        for (int j0 = 0; j0 < kTokens; j0 += PAIR) {
            if (j0 >= live) break;
            float wv[PAIR][NW], cv[PAIR][NW];
#pragma unroll
            for (int p = 0; p < PAIR; ++p) {
                const size_t row = w.rb + (tg + min(j0 + p, live - 1));
                load_row<NW>(c.Bm + row * N + w.ns, wv[p]);
                load_row<NW>(c.Cm + row * N + w.ns, cv[p]);
            }
#pragma unroll
            for (int p = 0; p < PAIR; ++p) {
                const int j = j0 + p;
                if (j >= live) break;
                float y2[2] = {0.f, 0.f};   // two sums, two dependency chains
#pragma unroll
                for (int n = 0; n < NW; ++n) {
                    const float dA = __builtin_amdgcn_exp2f(dl[j] * a2[n]);
                    const float z = u[j] * wv[p][n];
                    g[n] = __builtin_fmaf(dA, g[n] + z, -z);   // dA g + (dA - 1) z
                    y2[n & 1] = __builtin_fmaf(cv[p][n] * ia[n], g[n], y2[n & 1]);
                }
                acc[j] = y2[0] + y2[1];
                if constexpr (EARLY) w.store(c, c.y, tg + j, acc[j]);
                sd += dl[j];
            }
        }
        if constexpr (EARLY) return;
        add_shares<SPLIT, PER>(red[buf], w.wave, w.lane, acc);
        buf ^= 1;
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (PER * w.wave + j < live) w.store(c, c.y, tg + PER * w.wave + j, acc[j]);
    });
    if (w.ok()) {
        const int ch = w.channel();
        // A is read in full before any store (a store to the workspace could alias it, so
        // interleaved, every load would wait for the store before it)
        float a[NW];
#pragma unroll
        for (int n = 0; n < NW; ++n) a[n] = ap[n];
        float* hw = c.ws_h + (((size_t)w.b * c.nch + w.chunk) * c.d + ch) * N + w.ns;
#pragma unroll
        for (int n = 0; n < NW; ++n) hw[n] = g[n] / a[n];
        if (w.wave == 0) c.ws_s[((size_t)w.b * c.nch + w.chunk) * c.d + ch] = sd;
    }
}

// One thread per (batch entry, channel, state): the chunks' carries, in chunk order.
// One workgroup holds every segment of cpw = 256 / seg (channel, state) pairs of one batch
// entry: thread (segment s, pair j).  The chunks of a pair are split into seg consecutive
// segments; each thread scans its segment from zero (its chunks' values come in batches of
// kBatch loads issued before the recurrence, so one memory round trip per batch), the
// segments' end states and Delta sums meet in LDS, every thread combines those before its own
// (its carry in) and all of them (the state after one copy), and then runs over its segment
// again writing E_c = r H_{c-1} + P(start -> chunk c) G.  A segment of one batch keeps its
// values in registers for the second run.
__global__ __launch_bounds__(256) void cycle_scan_carries(CycleArgs c) {
    __shared__ float seg_h[256], seg_s[256];
    const int S = c.seg;
    const int cpw = 256 / S;
    const int tid = (int)threadIdx.x;
    const int j = tid % cpw, seg = tid / cpw;
    const long long per_b = (long long)c.d * c.N;
    const long long wg_per_b = (per_b + cpw - 1) / cpw;
    const int b = (int)(blockIdx.x / wg_per_b);
    const long long cn_ll = (long long)(blockIdx.x - b * wg_per_b) * cpw + j;
    const bool live = cn_ll < per_b;
    const int cn = live ? (int)cn_ll : (int)(per_b - 1);   // ch * N + n (past the end: a copy, not stored)
    const int ch = cn / c.N;
    const float a2 = c.A[cn] * kLog2e;
    const size_t hbase = (size_t)b * c.nch * per_b + cn;              // + chunk * d * N
    const size_t sbase = (size_t)b * c.nch * c.d + ch;                // + chunk * d
    const int cps = (c.nch + S - 1) / S;
    const int k_begin = min(seg * cps, c.nch), k_end = min(k_begin + cps, c.nch);
    const bool one_batch = k_end - k_begin <= kBatch;
    float sv[kBatch], hv[kBatch];
    auto load_batch = [&](int k0) {
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const int k = min(k0 + i, k_end - 1);
            sv[i] = c.ws_s[sbase + (size_t)k * c.d];
            hv[i] = c.ws_h[hbase + (size_t)k * per_b];
        }
    };
    // the segment from zero: its end state and the decay over it (as a sum of Delta)
    float H = 0.f, cum = 0.f;
    for (int k0 = k_begin; k0 < k_end; k0 += kBatch) {
        load_batch(k0);
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            if (k0 + i < k_end) {
                H = __builtin_fmaf(__builtin_amdgcn_exp2f(a2 * sv[i]), H, hv[i]);
                cum += sv[i];
            }
    }
    seg_h[tid] = H;
    seg_s[tid] = cum;
    __syncthreads();
    // the state entering this segment, and after the whole sequence (S_1) with its decay
    float Hin = 0.f, cin = 0.f, Htot = 0.f, ctot = 0.f;
    for (int s = 0; s < S; ++s) {
        if (s == seg) {
            Hin = Htot;
            cin = ctot;
        }
        const float cs = seg_s[s * cpw + j];
        Htot = __builtin_fmaf(__builtin_amdgcn_exp2f(a2 * cs), Htot, seg_h[s * cpw + j]);
        ctot += cs;
    }
    const float PL = __builtin_amdgcn_exp2f(a2 * ctot);
    float g = 0.f;   // sum_{i=0}^{r-2} (r-1-i) PL^i, Horner from the top power
    for (int i = c.repeats - 2; i >= 0; --i) g = __builtin_fmaf(g, PL, (float)(c.repeats - 1 - i));
    const float G = g * Htot;
    // E_c = r H_{c-1} + P(start -> chunk c) G over the segment's chunks
    H = Hin;
    cum = cin;
    const float r = (float)c.repeats;
    for (int k0 = k_begin; k0 < k_end; k0 += kBatch) {
        if (!one_batch) load_batch(k0);
#pragma unroll
        for (int i = 0; i < kBatch; ++i)
            if (k0 + i < k_end) {
                if (live)
                    c.ws_h[hbase + (size_t)(k0 + i) * per_b] = __builtin_fmaf(__builtin_amdgcn_exp2f(a2 * cum), G, r * H);
                H = __builtin_fmaf(__builtin_amdgcn_exp2f(a2 * sv[i]), H, hv[i]);
                cum += sv[i];
            }
    }
}

template <int N, int SPLIT>
__global__ __launch_bounds__(64 * SPLIT) __attribute__((amdgpu_waves_per_eu(1, N == 32 && SPLIT == 1 ? 3 : 8)))
void cycle_scan_outputs(CycleArgs c) {
    using W = ScanWave<N, SPLIT>;
    constexpr int NW = W::NW, PER = W::PER, PAIR = W::PAIR;
    __shared__ float red[2][SPLIT][kTokens][64];
    const W w(c);
    const float* ap = c.A + (size_t)w.channel() * N + w.ns;
    const float* hw = c.ws_h + (((size_t)w.b * c.nch + w.chunk) * c.d + w.channel()) * N + w.ns;
    float a2[NW], e[NW];
#pragma unroll
    for (int n = 0; n < NW; ++n) {
        a2[n] = ap[n] * kLog2e;
        e[n] = hw[n];   // E_c
    }
    const float r = (float)c.repeats;
    float cum = 0.f;   // sum of Delta from the chunk's start to t
    int buf = 0;
    for_groups(w.t0, w.t1, [&](int tg, auto live) {
        float dl[kTokens], y1[PER], acc[kTokens];
#pragma unroll
        for (int j = 0; j < kTokens; ++j) {
            dl[j] = acc[j] = 0.f;
            if (j < live) dl[j] = w.load(c, c.delta, tg + j);
        }
#pragma unroll
        for (int j = 0; j < PER; ++j)   // the tokens this wave stores
            y1[j] = PER * w.wave + j < live ? w.load(c, c.y, tg + PER * w.wave + j) : 0.f;
#pragma unroll
        for (int j0 = 0; j0 < kTokens; j0 += PAIR) {
            if (j0 >= live) break;
            float cv[PAIR][NW];
#pragma unroll
            for (int p = 0; p < PAIR; ++p)
                load_row<NW>(c.Cm + (w.rb + (tg + min(j0 + p, live - 1))) * N + w.ns, cv[p]);
#pragma unroll
            for (int p = 0; p < PAIR; ++p) {
                const int j = j0 + p;
                if (j >= live) break;
                cum += dl[j];
                float y2[2] = {0.f, 0.f};
#pragma unroll
                for (int n = 0; n < NW; ++n) {
                    const float dec = __builtin_amdgcn_exp2f(a2[n] * cum);   // decay from the chunk's start
                    y2[n & 1] = __builtin_fmaf(cv[p][n], dec * e[n], y2[n & 1]);
                }
                acc[j] = y2[0] + y2[1];
            }
        }
        add_shares<SPLIT, PER>(red[buf], w.wave, w.lane, acc);
        buf ^= 1;
        // each lane reads y1 and then writes y at its own address
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if (PER * w.wave + j < live) w.store(c, c.y, tg + PER * w.wave + j, __builtin_fmaf(r, y1[j], acc[j]));
    });
}

// SPA, SPC: waves per group of passes A and C
template <int N, int SPA, int SPC, bool EARLY = false>
hipError_t launch_n(const CycleArgs& a, hipStream_t stream) {
    CycleArgs args = a;
    // carry pass: up to 8 segments of at least kBatch chunks per (channel, state)
    args.seg = 1;
    while (args.seg < 8 && (long long)args.seg * kBatch < a.nch) args.seg *= 2;
    void* params[] = {&args};
    const long long scan_groups = (long long)a.B * a.nch * a.cgroups;
    hipError_t e = hipLaunchKernel(reinterpret_cast<const void*>(&cycle_scan_chunks<N, SPA, EARLY>),
                                   dim3((unsigned)scan_groups), dim3(64 * SPA), params, 0, stream);
    if (e != hipSuccess) return e;
    const long long per_wg = 256 / args.seg;
    const long long carry_groups = (long long)a.B * (((long long)a.d * a.N + per_wg - 1) / per_wg);
    e = hipLaunchKernel(reinterpret_cast<const void*>(&cycle_scan_carries), dim3((unsigned)carry_groups), dim3(256),
                        params, 0, stream);
    if (e != hipSuccess) return e;
    return hipLaunchKernel(reinterpret_cast<const void*>(&cycle_scan_outputs<N, SPC>), dim3((unsigned)scan_groups),
                           dim3(64 * SPC), params, 0, stream);
}

}  // namespace

bool cycle_states_supported(int N) { return N == 1 || N == 2 || N == 4 || N == 8 || N == 16 || N == 32; }

hipError_t launch_cycle_scan(const CycleArgs& a, hipStream_t stream) {
    // Waves that share one chunk's states, by the number of (chunk, 64 channels) groups; the numbers are
    // those of 256 compute units, 1024 SIMDs.  Few groups leave SIMDs without a wave (one wave alone
    // issues at half the rate of two): more waves per group, as long as six per SIMD hold them all
    // (1536 groups of four waves).  Many: fewer, since every wave reads the group's x and Delta and joins
    // the sum.  Up to 8 states one wave holds them all.  Measured per call, us, by waves in pass A / C
    // (chunks of 256 tokens unless said; "early": see cycle_scan_chunks):
    //   32 states  8/8 and 4/4: 768 groups (chunks of 64) 72, 73.  4/4 and 4/1: 1536 groups 375, 406;
    //     1884 476, 531; 2160 541, 561; 2448 585, 596; 2820 634, 633; 3060 676, 662; 3072 681, 666; 3288 733,
    //     787; 4104 871, 881; 4608 979, 997; 5640 1163, 1187; 6144 1255, 1245; 8192 1653, 1630.  1/1 is slower
    //     throughout (3072: 718).
    //   16 states  4/4, 2/1, 1/1: 948 groups 188, 231, 237; 1416 240, 246, 273; 1536 248, 268, 287; 1548 306, 269,
    //     287; 1884 352, 329, 312; 2160 393, 336, 366; 2448 418, 362, 380; 2820 452, 380, 392; 3060 469, 405, 400;
    //     3288 554, 473, 459; 4608 700, 579, 552.  2/2 lies between 2/1 and 4/4 up to 3060 groups and is slower
    //     than 2/1 from there (4608: 682).  1/1 and 1/1 early: 4608 groups 552, 554; 5640 679, 637; 6144 716, 662,
    //     in chunks of 64 194, 181; 8192 897, 922: early where six waves per SIMD hold all groups and five do not.
    const long long groups = (long long)a.B * a.nch * a.cgroups;
    switch (a.N) {
        case 1: return launch_n<1, 1, 1>(a, stream);
        case 2: return launch_n<2, 1, 1>(a, stream);
        case 4: return launch_n<4, 1, 1>(a, stream);
        case 8: return launch_n<8, 1, 1>(a, stream);
        case 16:
            return groups <= 1536                     ? launch_n<16, 4, 4>(a, stream)
                   : groups <= 3072                   ? launch_n<16, 2, 1>(a, stream)
                   : groups > 5120 && groups <= 6144 ? launch_n<16, 1, 1, true>(a, stream)
                                                      : launch_n<16, 1, 1>(a, stream);
        case 32:
            return groups >= 2816   ? launch_n<32, 4, 1>(a, stream)
                   : groups >= 1024 ? launch_n<32, 4, 4>(a, stream)
                                    : launch_n<32, 8, 8>(a, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fla

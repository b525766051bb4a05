// Chunkwise-parallel mLSTM forward, fp32, for small heads: an fp64-MFMA kernel for head sizes that are
// multiples of 16 with chunks of 16, 32 or 64 tokens, and a VALU kernel for every other size.
//
// The chunkwise form (Sec. 2, "Training Mode") processes the sequence in
// chunks of L tokens: within a chunk the outputs come from a causal,
// gate-weighted L x L matrix (the intra-chunk part), and the chunk's entry
// state carries everything before it (the inter-chunk part).  The sub-steps
// follow App. D.1: chunkwise gates (prefix sums of logsig f~), gates and max
// state, inter-chunk numerator and denominator, gate matrix, gated logits,
// intra-chunk numerator and denominator, output combination.
//
// Stabiliser bookkeeping.  With b_tau the in-chunk prefix sum of logsig f~
// and p_tau = max_{sig <= tau}(i~_sig - b_sig), the max state of Eq. 2 is
// m_tau = b_tau + M_tau with M_tau = max(m_prev, p_tau).  Every exponent is
// then written as a difference against M, so it is <= 0 by construction:
//   gate matrix      D[tau,sig] = exp((i~_sig - b_sig) - M_tau)     (sig <= tau)
//   entry-state term             exp(m_prev - M_tau)
//   state decay                  exp(m_prev - M_L)
//   key weights      w_tau     = exp((i~_tau - b_tau) - M_L)
//   floor                        exp(-(b_tau + M_tau))
// and the chunk's exit max state is b_L + M_L.
//
// A forget gate of exactly zero (f~ = -inf, a document border) restarts the state.  The prefix
// sum b skips the restart token, each row keeps its last restart R_tau, the gate matrix keeps
// only R_tau <= sig <= tau, p restarts at R_tau, a row at or after a restart has no entry-state
// term, and a chunk that holds a restart drops its entry state (decay 0) and weights only the
// keys from its last restart on.
//
// One workgroup owns a (sequence, dv tile) pair and walks the chunks in order with its C tile, n and m.
// q, k, v may be fp32 or bf16; the gate matrix is fp32.  The dot products (logits, read-outs, state
// updates) accumulate in fp64, so a row whose sum cancels keeps the accuracy of its fp32 operands rather
// than of an fp32 sum.  This is the fp32 path; the bf16 xLSTM-7B head shape runs on the bf16 MFMA kernel.
#include "launch.h"
#include "mfma_common.h"

namespace mlstm {

constexpr int kF32Threads = 256;
constexpr size_t kF32LdsBudget = 64 * 1024;

static size_t f32_lds_floats(int DQK, int DVT, int L) {
    return static_cast<size_t>(DQK) * DVT + DQK + 2 * static_cast<size_t>(L) * DQK +
           static_cast<size_t>(L) * DVT + static_cast<size_t>(L) * L + 8 * static_cast<size_t>(L) + 8;
}

int chunk_f32_tile(int DQK, int DV, int L) {
    for (int dvt = DV; dvt >= 1; dvt >>= 1) {
        if (DV % dvt) continue;
        if (f32_lds_floats(DQK, dvt, L) * sizeof(float) <= kF32LdsBudget) return dvt;
        if (dvt & 1) break;
    }
    return 0;
}

template <typename TIn>
__global__ void __launch_bounds__(kF32Threads)
chunk_f32_kernel(const TIn* __restrict__ q, const TIn* __restrict__ k, const TIn* __restrict__ v,
                 const float* __restrict__ ipre, const float* __restrict__ fpre,
                 const float* __restrict__ C0, const float* __restrict__ n0, const float* __restrict__ m0,
                 int T, int DQK, int DV, int L, int DVT, TIn* __restrict__ h, float* __restrict__ CT,
                 float* __restrict__ nT, float* __restrict__ mT) {
    extern __shared__ float smem[];
    float* Cs = smem;                                   // [DQK][DVT]
    float* ns = Cs + DQK * DVT;                         // [DQK]
    float* Qs = ns + DQK;                               // [L][DQK]   q / sqrt(DQK)
    float* Ks = Qs + L * DQK;                           // [L][DQK]
    float* Vs = Ks + L * DQK;                           // [L][DVT]
    float* Sm = Vs + L * DVT;                           // [L][L]     gated logits S~
    float* g_ib = Sm + L * L;                           // [L]  i~ - b
    float* g_M = g_ib + L;                              // [L]  M_tau
    float* g_inter = g_M + L;                           // [L]  exp(m_prev - M_tau)
    float* g_floor = g_inter + L;                       // [L]  exp(-(b_tau + M_tau))
    float* g_w = g_floor + L;                           // [L]  key weights
    float* g_den = g_w + L;                             // [L]  1 / max(|den|, floor)
    float* g_sc = g_den + 2 * L;                        // scalars: [0] m_prev, [1] decay
    float* g_R = g_sc + 8;                              // [L]  last restart at or before the row (-1: none)

    const int ntiles = DV / DVT;
    const int64_t seq = blockIdx.x / ntiles;
    const int tile = blockIdx.x % ntiles;
    MLSTM_CHECK(ntiles * DVT == DV && L <= T + L, kDbgChunkF32);
    const int v0 = tile * DVT;
    const int tid = threadIdx.x;
    const float qscale = rsqrtf(static_cast<float>(DQK));

    // initial state (zero state has m0 = 0)
    for (int e = tid; e < DQK * DVT; e += kF32Threads) {
        const int d = e / DVT, j = e % DVT;
        Cs[e] = C0 ? C0[(seq * DQK + d) * DV + v0 + j] : 0.0f;
    }
    for (int d = tid; d < DQK; d += kF32Threads) ns[d] = n0 ? n0[seq * DQK + d] : 0.0f;
    if (tid == 0) g_sc[0] = m0 ? m0[seq] : 0.0f;
    __syncthreads();

    const TIn* qb = q + seq * static_cast<int64_t>(T) * DQK;
    const TIn* kb = k + seq * static_cast<int64_t>(T) * DQK;
    const TIn* vb = v + seq * static_cast<int64_t>(T) * DV;
    TIn* hb = h + seq * static_cast<int64_t>(T) * DV;

    for (int t0 = 0; t0 < T; t0 += L) {
        // rows lc..L-1 of a partial last chunk are neutral tokens: zero q, k, v, no input
        // (x = -inf) and no decay, so they leave the state unchanged; their h is not written
        const int lc = min(L, T - t0);
        // stage the chunk
        for (int e = tid; e < L * DQK; e += kF32Threads) {
            const bool ok = e < lc * DQK;
            Qs[e] = ok ? io<TIn>::load(qb, static_cast<int64_t>(t0) * DQK + e) * qscale : 0.0f;
            Ks[e] = ok ? io<TIn>::load(kb, static_cast<int64_t>(t0) * DQK + e) : 0.0f;
        }
        for (int e = tid; e < L * DVT; e += kF32Threads) {
            const int t = e / DVT, j = e % DVT;
            Vs[e] = t < lc ? io<TIn>::load(vb, static_cast<int64_t>(t0 + t) * DV + v0 + j) : 0.0f;
        }
        // chunkwise gates and max state: a short serial scan (L <= 64)
        if (tid == 0) {
            const float mprev = g_sc[0];
            const float* ib = ipre + seq * static_cast<int64_t>(T) + t0;
            const float* fb = fpre + seq * static_cast<int64_t>(T) + t0;
            float b = 0.0f, p = -INFINITY;
            int R = -1;
            for (int t = 0; t < L; ++t) {
                const float lg = t < lc ? logsigmoid(fb[t]) : 0.0f;
                if (lg == -INFINITY) {
                    R = t;
                    p = -INFINITY;
                } else {
                    b += lg;
                }
                const float x = t < lc ? ib[t] - b : -INFINITY;
                p = fmaxf(p, x);
                const float M = R >= 0 ? p : fmaxf(mprev, p);
                g_ib[t] = x;
                g_M[t] = M;
                g_R[t] = static_cast<float>(R);
                g_inter[t] = (R >= 0 || M == -INFINITY) ? 0.0f : expf(mprev - M);
                g_floor[t] = expf(-(b + M));
            }
            const float ML = g_M[L - 1];
            for (int t = 0; t < L; ++t) g_w[t] = (t < R || ML == -INFINITY) ? 0.0f : expf(g_ib[t] - ML);
            g_sc[1] = (R >= 0 || ML == -INFINITY) ? 0.0f : expf(mprev - ML);
            g_sc[0] = b + ML;  // exit max state m_k
        }
        __syncthreads();

        // gated logits S~ = (Q^ K^T) * D, causal
        for (int e = tid; e < L * L; e += kF32Threads) {
            const int t = e / L, s = e % L;
            float val = 0.0f;
            if (s <= t && s >= static_cast<int>(g_R[t]) && g_M[t] != -INFINITY) {
                double acc = 0.0;
                for (int d = 0; d < DQK; ++d) acc += static_cast<double>(Qs[t * DQK + d]) * Ks[s * DQK + d];
                val = static_cast<float>(acc) * expf(g_ib[s] - g_M[t]);
            }
            Sm[e] = val;
        }
        __syncthreads();

        // denominators: exp(m_prev - M) q^.n + rowsum(S~), floored
        for (int t = tid; t < L; t += kF32Threads) {
            double qn = 0.0;
            for (int d = 0; d < DQK; ++d) qn += static_cast<double>(Qs[t * DQK + d]) * ns[d];
            double rs = 0.0;
            for (int s = 0; s <= t; ++s) rs += Sm[t * L + s];
            const float den = static_cast<float>(g_inter[t] * qn + rs);
            g_den[t] = 1.0f / fmaxf(fabsf(den), g_floor[t]);
        }
        __syncthreads();

        // numerators and output combination
        for (int e = tid; e < lc * DVT; e += kF32Threads) {
            const int t = e / DVT, j = e % DVT;
            double inter = 0.0;
            for (int d = 0; d < DQK; ++d) inter += static_cast<double>(Qs[t * DQK + d]) * Cs[d * DVT + j];
            double intra = 0.0;
            for (int s = 0; s <= t; ++s) intra += static_cast<double>(Sm[t * L + s]) * Vs[s * DVT + j];
            io<TIn>::store(hb, static_cast<int64_t>(t0 + t) * DV + v0 + j,
                           static_cast<float>((g_inter[t] * inter + intra) * g_den[t]));
        }
        __syncthreads();

        // state update: C = decay C + (w K)^T V, n = decay n + K^T w
        const float decay = g_sc[1];
        for (int e = tid; e < DQK * DVT; e += kF32Threads) {
            const int d = e / DVT, j = e % DVT;
            double acc = 0.0;
            for (int t = 0; t < L; ++t) acc += static_cast<double>(g_w[t] * Ks[t * DQK + d]) * Vs[t * DVT + j];
            Cs[e] = static_cast<float>(decay * static_cast<double>(Cs[e]) + acc);
        }
        for (int d = tid; d < DQK; d += kF32Threads) {
            double acc = 0.0;
            for (int t = 0; t < L; ++t) acc += static_cast<double>(g_w[t]) * Ks[t * DQK + d];
            ns[d] = static_cast<float>(decay * static_cast<double>(ns[d]) + acc);
        }
        __syncthreads();
    }

    // final state
    for (int e = tid; e < DQK * DVT; e += kF32Threads) {
        const int d = e / DVT, j = e % DVT;
        CT[(seq * DQK + d) * DV + v0 + j] = Cs[e];
    }
    if (tile == 0) {
        for (int d = tid; d < DQK; d += kF32Threads) nT[seq * DQK + d] = ns[d];
        if (tid == 0) mT[seq] = g_sc[0];
    }
}

// ---- fp64 MFMA kernel ---------------------------------------------------------------------------
// A chunk is a short serial step (32 of them for 512 tokens at L = 16), so its latency bounds the kernel and
// the work is spread for that: one workgroup of four waves per (sequence, 16 columns of dv), with the
// products on 16x16x4 fp64 MFMA (one LDS read per operand lane and 16 FMAs, where the VALU kernel reads two
// operands from LDS per FMA) and the gates as scans over the lanes of one wave (the VALU kernel's scan is
// serial in one thread).  8 sequences of 512 tokens, heads of 64 x 128, L = 16: 87 us, 2.7 us a
// chunk (the VALU kernel: 2512 us).
//
// MFMA mapping: lane (l16, g) holds A[m = l16][k = g], B[k = g][n = l16] and receives D[m = 4 i + g]
// [n = l16] in its i-th value, so the state tiles, kept as D in fp64 registers, are the B operands of the
// read-out C^T q as they stand.  Wave w owns the 16-row tiles w, w + 4, ... of C: its partial read-outs are
// summed over the waves in LDS, and so are (L = 16, one tile of S) its partial logits; with longer chunks
// the tiles of S go to the waves whole.
typedef double f64x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f64x4_t mfma_f64(double a, double b, f64x4_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
// fp64 values across lanes with DPP (a shuffle of two words through LDS takes a few hundred cycles, and a
// chunk's serial path had twenty of them: 114 us became 92).
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_f64(double x) {   // lanes without a source: 0
    const uint64_t u = __builtin_bit_cast(uint64_t, x);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u), kCtrl, kRowMask, 0xf, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), kCtrl, kRowMask, 0xf, false);
    return __builtin_bit_cast(double, (static_cast<uint64_t>(hi) << 32) | lo);
}
__device__ __forceinline__ double wave_incl_sum_f64(double x) {   // inclusive prefix sum over the 64 lanes
    x += dpp_f64<0x111, 0xf>(x);   // row_shr:1
    x += dpp_f64<0x112, 0xf>(x);   // row_shr:2
    x += dpp_f64<0x114, 0xf>(x);   // row_shr:4
    x += dpp_f64<0x118, 0xf>(x);   // row_shr:8
    x += dpp_f64<0x142, 0xa>(x);   // row_bcast:15 into rows 1 and 3
    x += dpp_f64<0x143, 0xc>(x);   // row_bcast:31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ double row_sum_f64(double x) {   // sum over 16 lanes, in each of them
    x += dpp_f64<0xB1, 0xf>(x);    // quad_perm [1, 0, 3, 2]
    x += dpp_f64<0x4E, 0xf>(x);    // quad_perm [2, 3, 0, 1]
    x += dpp_f64<0x141, 0xf>(x);   // row_half_mirror
    x += dpp_f64<0x140, 0xf>(x);   // row_mirror
    return x;
}
__device__ __forceinline__ float lane_f32(float x, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), l));
}
__device__ __forceinline__ float4 load4f(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ float4 load4f(const bf16_t* p) {
    const uint2 u = *reinterpret_cast<const uint2*>(p);
    return make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                       __uint_as_float(u.y & 0xffff0000u));
}

struct F32Args {
    const void* q;
    const void* k;
    const void* v;
    const float* ipre;
    const float* fpre;
    const float* C0;
    const float* n0;
    const float* m0;
    int T, DQK, DV;
    void* h;
    float* CT;
    float* nT;
    float* mT;
};

constexpr int kMmaW = 4;          // waves
constexpr int kMmaVP = 16 + 4;    // row pitch of V (floats)
// LDS of the kernel (bytes): partial read-outs, partial logits (L = 16), n, q . n and 1 / den in fp64, then
// Q, K, V, S and two buffers of six gate rows in fp32
size_t f32_mma_lds(int DQK, int L) {
    const size_t d = kMmaW * static_cast<size_t>(L) * 16 + (L == 16 ? kMmaW * 256 : 0) + DQK + 2 * static_cast<size_t>(L);
    const size_t f = 2 * static_cast<size_t>(L) * (DQK + 4) + static_cast<size_t>(L) * kMmaVP +
                     static_cast<size_t>(L) * (L + 4) + 2 * (6 * static_cast<size_t>(L) + 4);
    return d * sizeof(double) + f * sizeof(float);
}

// TPW: 16-row tiles of C per wave, DQK <= 64 TPW
template <typename TIn, int L, int TPW>
__global__ void __launch_bounds__(64 * kMmaW) chunk_f32_mma_kernel(F32Args A) {
    extern __shared__ double smem_d[];
    constexpr int NT = L / 16, NTHR = 64 * kMmaW;
    constexpr int kGw = NT == kMmaW ? 0 : kMmaW - 1;            // the wave of the gates
    constexpr int NLD = (L * 64 * TPW / 4 + NTHR - 1) / NTHR;   // 4-element pieces of q (and of k) per thread
    const int DQK = A.DQK, DV = A.DV, T = A.T;
    const int QP = DQK + 4, SP = L + 4;
    double* Np = smem_d;                                  // [kMmaW][L][16] partial read-outs
    double* Sp = Np + kMmaW * L * 16;                     // [kMmaW][16][16] partial logits (L = 16)
    double* ns = Sp + (L == 16 ? kMmaW * 256 : 0);        // [DQK]
    double* qn = ns + DQK;                                // [L] q . n
    double* inv = qn + L;                                 // [L] 1 / max(|den|, floor)
    float* Qs = reinterpret_cast<float*>(inv + L);        // [L][QP]
    float* Ks = Qs + L * QP;                              // [L][QP]
    float* Vs = Ks + L * QP;                              // [L][kMmaVP]
    float* Sm = Vs + L * kMmaVP;                          // [L][SP] gated logits
    float* gates = Sm + L * SP;                           // [2][6 L + 4] by chunk parity, see below

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g = lane >> 4;
    const int ntile = DV / 16;
    const int64_t seq = blockIdx.x / ntile;
    const int v0 = 16 * static_cast<int>(blockIdx.x % ntile);
    const int ndt = DQK / 16;
    const double qscale = 1.0 / sqrt(static_cast<double>(DQK));
    const TIn* qb = static_cast<const TIn*>(A.q) + seq * T * DQK;
    const TIn* kb = static_cast<const TIn*>(A.k) + seq * T * DQK;
    const TIn* vb = static_cast<const TIn*>(A.v) + seq * T * DV + v0;
    TIn* hb = static_cast<TIn*>(A.h) + seq * T * DV + v0;
    MLSTM_CHECK(DQK <= 64 * TPW && DQK % 16 == 0 && v0 + 16 <= DV, kDbgChunkF32);

    f64x4_t C[TPW];
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
        const int dt = wave + kMmaW * u;
        C[u] = f64x4_t{0.0, 0.0, 0.0, 0.0};
        if (A.C0 && dt < ndt)
#pragma unroll
            for (int i = 0; i < 4; ++i) C[u][i] = A.C0[(seq * DQK + 16 * dt + 4 * i + g) * DV + v0 + l16];
    }
    for (int d = tid; d < DQK; d += NTHR) ns[d] = A.n0 ? A.n0[seq * DQK + d] : 0.0f;
    float m_prev = A.m0 ? A.m0[seq] : 0.0f;

    // one chunk of inputs in registers; rows past the end are zero
    const int qk4 = DQK / 4;   // pieces per row
    float4 rq[NLD], rk[NLD], rv;
    float gi = 0.0f, gf = 0.0f;
    auto load = [&](int t0) {
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int e = tid + NTHR * i, t = t0 + e / qk4;
            rq[i] = rk[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (e < L * qk4 && t < T) {
                rq[i] = load4f(qb + static_cast<int64_t>(t) * DQK + 4 * (e % qk4));
                rk[i] = load4f(kb + static_cast<int64_t>(t) * DQK + 4 * (e % qk4));
            }
        }
        rv = make_float4(0.f, 0.f, 0.f, 0.f);
        if (tid < 4 * L && t0 + tid / 4 < T) rv = load4f(vb + static_cast<int64_t>(t0 + tid / 4) * DV + 4 * (tid % 4));
        if (wave == kGw && lane < L && t0 + lane < T) {
            gi = A.ipre[seq * T + t0 + lane];
            gf = A.fpre[seq * T + t0 + lane];
        }
    };
    // One wave computes the gates of a chunk while another finishes the chunk before: with L = 16 or 32 the
    // last wave, which has no tile of h; with L = 64 the first, whose tile has the fewest products.
    auto compute_gates = [&](int t0, float* gb) {
        float *g_x = gb, *g_M = gb + L, *g_inter = gb + 2 * L, *g_floor = gb + 3 * L, *g_w = gb + 4 * L, *g_sc = gb + 6 * L;
        int* g_R = reinterpret_cast<int*>(gb + 5 * L);
        // gates and max state, one token per lane (lanes from L on are neutral tokens as well)
        const bool ok = lane < min(L, T - t0);
        const float lg = ok ? logsigmoid(gf) : 0.0f;
        const bool rs = (lg == -INFINITY);
        const bool any_restart = __builtin_amdgcn_ballot_w64(rs) != 0;   // rare; wave-uniform
        const double b = wave_incl_sum_f64(rs ? 0.0 : static_cast<double>(lg));
        const float x = ok ? static_cast<float>(static_cast<double>(gi) - b) : -INFINITY;
        int R = -1;
        float pm;           // maximum of x from the last restart on
        if (any_restart) {
            R = static_cast<int>(wave_incl_max(rs ? static_cast<float>(lane) : -1.0f));
            pm = wave_seg_incl_max(x, rs);
        } else {
            pm = wave_incl_max(x);
        }
        const float M = R >= 0 ? pm : fmaxf(m_prev, pm);
        const float ML = lane_f32(M, L - 1);
        const int RL = __builtin_amdgcn_readlane(R, L - 1);
        const uint64_t bu = __builtin_bit_cast(uint64_t, b);
        const double bL = __builtin_bit_cast(
            double, (static_cast<uint64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(bu >> 32), L - 1))) << 32) |
                        static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(bu), L - 1)));
        if (lane < L) {
            g_x[lane] = x;
            g_M[lane] = M;
            g_R[lane] = R;
            g_inter[lane] = (R >= 0 || M == -INFINITY) ? 0.0f : expf(m_prev - M);
            g_floor[lane] = expf(static_cast<float>(-(b + M)));
            g_w[lane] = (lane < RL || ML == -INFINITY) ? 0.0f : expf(x - ML);
        }
        if (lane == 0) g_sc[0] = (RL >= 0 || ML == -INFINITY) ? 0.0f : expf(m_prev - ML);
        m_prev = static_cast<float>(bL + ML);
    };
    if (T > 0) {
        load(0);
        if (wave == kGw) compute_gates(0, gates);
    }

    int par = 0;
    for (int t0 = 0; t0 < T; t0 += L, par ^= 1) {
        const float* gb = gates + par * (6 * L + 4);   // i~ - b, M, scales of the entry state, floors, key weights
        const float *g_x = gb, *g_M = gb + L, *g_inter = gb + 2 * L, *g_floor = gb + 3 * L, *g_w = gb + 4 * L;
        const int* g_R = reinterpret_cast<const int*>(gb + 5 * L);   // last restart at or before the row
        const float* g_sc = gb + 6 * L;                              // decay
        const int lc = min(L, T - t0);
        __syncthreads();   // the previous chunk's readers are done
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int e = tid + NTHR * i;
            if (e < L * qk4) {
                const int off = (e / qk4) * QP + 4 * (e % qk4);
                *reinterpret_cast<float4*>(&Qs[off]) = rq[i];
                *reinterpret_cast<float4*>(&Ks[off]) = rk[i];
            }
        }
        if (tid < 4 * L) *reinterpret_cast<float4*>(&Vs[(tid / 4) * kMmaVP + 4 * (tid % 4)]) = rv;
        if (t0 + L < T) load(t0 + L);
        __syncthreads();   // the chunk and its gates are visible

        // read-out partials over this wave's rows of C, with (L = 16) the logits over the same rows
        f64x4_t N[NT], Sa = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) N[nt] = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
            const int dt = wave + kMmaW * u;
            if (dt < ndt) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int d = 16 * dt + 4 * i + g;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const double a = Qs[(16 * nt + l16) * QP + d];
                        N[nt] = mfma_f64(a, C[u][i], N[nt]);
                        if constexpr (L == 16) Sa = mfma_f64(a, Ks[l16 * QP + d], Sa);
                    }
                }
            }
        }
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int i = 0; i < 4; ++i) Np[(wave * L + 16 * nt + 4 * i + g) * 16 + l16] = N[nt][i];
        auto gated = [&](double acc, int t, int s2) {
            return (s2 <= t && s2 >= g_R[t] && g_M[t] != -INFINITY)
                       ? static_cast<float>(acc * qscale) * expf(g_x[s2] - g_M[t]) : 0.0f;
        };
        if constexpr (L == 16) {
#pragma unroll
            for (int i = 0; i < 4; ++i) Sp[wave * 256 + (4 * i + g) * 16 + l16] = Sa[i];
        } else {
            // causal tiles of S, whole, one after another to the waves; the tiles above the diagonal are zero
            int idx = 0;
            for (int tb = 0; tb < NT; ++tb)
                for (int sb = 0; sb < NT; ++sb, ++idx) {
                    if ((idx & (kMmaW - 1)) != wave) continue;
                    f64x4_t acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
                    if (sb <= tb)
                        for (int k4 = 0; k4 < DQK; k4 += 4)
                            acc = mfma_f64(Qs[(16 * tb + l16) * QP + k4 + g], Ks[(16 * sb + l16) * QP + k4 + g], acc);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int t = 16 * tb + 4 * i + g, s2 = 16 * sb + l16;
                        Sm[t * SP + s2] = gated(acc[i], t, s2);
                    }
                }
        }
        // q . n: 16 lanes per row
        for (int t = tid >> 4; t < L; t += NTHR / 16) {
            double acc = 0.0;
            for (int d = l16; d < DQK; d += 16) acc += static_cast<double>(Qs[t * QP + d]) * ns[d];
            acc = row_sum_f64(acc);
            if (l16 == 0) qn[t] = acc * qscale;
        }
        __syncthreads();   // partials, q . n and (L > 16) S are visible; n is read

        // S (L = 16: the sum of the partials, gated), its row sums, 1 / max(|den|, floor)
        for (int t = tid >> 4; t < L; t += NTHR / 16) {
            double rs = 0.0;
            for (int s2 = l16; s2 < L; s2 += 16) {
                float val;
                if constexpr (L == 16) {
                    const int e = t * 16 + s2;
                    val = gated((Sp[e] + Sp[256 + e]) + (Sp[512 + e] + Sp[768 + e]), t, s2);
                    Sm[t * SP + s2] = val;
                } else {
                    val = Sm[t * SP + s2];
                }
                rs += val;
            }
            rs = row_sum_f64(rs);
            if (l16 == 0) inv[t] = 1.0 / fmax(fabs(static_cast<double>(g_inter[t]) * qn[t] + rs), static_cast<double>(g_floor[t]));
        }
        // C = decay C + (w K)^T V on this wave's tiles, n = decay n + K^T w
        const double decay = g_sc[0];
#pragma unroll
        for (int u = 0; u < TPW; ++u) {
            const int dt = wave + kMmaW * u;
            if (dt < ndt) {
                C[u] *= decay;
                for (int t4 = 0; t4 < L; t4 += 4) {
                    const int t = t4 + g;
                    C[u] = mfma_f64(static_cast<double>(g_w[t]) * Ks[t * QP + 16 * dt + l16], Vs[t * kMmaVP + l16], C[u]);
                }
            }
        }
        for (int d = tid >> 2; d < DQK; d += NTHR / 4) {   // four lanes per element
            double acc = 0.0;
#pragma unroll
            for (int t = 0; t < L; t += 4) acc += static_cast<double>(g_w[t + (tid & 3)]) * Ks[(t + (tid & 3)) * QP + d];
            acc += dpp_f64<0xB1, 0xf>(acc);   // quad_perm [1, 0, 3, 2]
            acc += dpp_f64<0x4E, 0xf>(acc);   // quad_perm [2, 3, 0, 1]
            if ((tid & 3) == 0) ns[d] = decay * ns[d] + acc;
        }
        __syncthreads();   // S and 1 / den are visible

        if (wave == kGw && t0 + L < T) compute_gates(t0 + L, gates + (par ^ 1) * (6 * L + 4));
        // h = (inter N + S V) / den
        for (int nt = wave; nt < NT; nt += kMmaW) {
            f64x4_t acc;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int t = 16 * nt + 4 * i + g;
                double sum = 0.0;
#pragma unroll
                for (int w = 0; w < kMmaW; ++w) sum += Np[(w * L + t) * 16 + l16];
                acc[i] = static_cast<double>(g_inter[t]) * qscale * sum;
            }
            for (int s4 = 0; s4 < 16 * nt; s4 += 4)
                acc = mfma_f64(Sm[(16 * nt + l16) * SP + s4 + g], Vs[(s4 + g) * kMmaVP + l16], acc);
            float vd[4];   // the diagonal tile, zero in S above the diagonal
            bool finite = true;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                vd[i] = Vs[(16 * nt + 4 * i + g) * kMmaVP + l16];
                finite = finite && fabsf(vd[i]) < INFINITY;
            }
            if (__builtin_amdgcn_ballot_w64(finite) == ~uint64_t{0}) {
#pragma unroll
                for (int i = 0; i < 4; ++i) acc = mfma_f64(Sm[(16 * nt + l16) * SP + 16 * nt + 4 * i + g], vd[i], acc);
            } else {   // zero times inf or NaN would reach the tokens before it: only the terms s <= t
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    for (int r = 0; r <= 4 * i + g; ++r)
                        acc[i] += static_cast<double>(Sm[(16 * nt + 4 * i + g) * SP + 16 * nt + r]) * Vs[(16 * nt + r) * kMmaVP + l16];
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int t = 16 * nt + 4 * i + g;
                if (t < lc) io<TIn>::store(hb, static_cast<int64_t>(t0 + t) * DV + l16, static_cast<float>(acc[i] * inv[t]));
            }
        }
    }
    __syncthreads();

#pragma unroll
    for (int u = 0; u < TPW; ++u) {
        const int dt = wave + kMmaW * u;
        if (dt < ndt)
#pragma unroll
            for (int i = 0; i < 4; ++i) A.CT[(seq * DQK + 16 * dt + 4 * i + g) * DV + v0 + l16] = static_cast<float>(C[u][i]);
    }
    if (v0 == 0) {
        for (int d = tid; d < DQK; d += NTHR) A.nT[seq * DQK + d] = static_cast<float>(ns[d]);
        if (tid == 64 * kGw) A.mT[seq] = m_prev;
    }
}

template <typename TIn, int L, int TPW>
hipError_t launch_f32_mma(const F32Args& a, int S, hipStream_t stream) {
    static std::atomic<uint64_t> raised{0};
    auto kern = chunk_f32_mma_kernel<TIn, L, TPW>;
    const size_t lds = f32_mma_lds(a.DQK, L);
    // the largest this instance can be asked for: the limit is raised once per device
    hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(kern), f32_mma_lds(64 * TPW, L), raised);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(S * (a.DV / 16))), dim3(64 * kMmaW), lds, stream, a);
    return hipGetLastError();
}
// The fp64-MFMA kernel's sizes: multiples of 16, and an LDS footprint within the CU's 160 KB (every size the
// VALU kernel takes with L = 16, 32 or 64 fits).
bool f32_mma_supported(int DQK, int DV, int L) {
    return DQK % 16 == 0 && DV % 16 == 0 && (L == 16 || L == 32 || L == 64) && DQK <= (L == 16 ? 512 : L == 32 ? 256 : 128) &&
           f32_mma_lds(L == 16 && DQK > 256 ? 512 : DQK > 128 ? 256 : DQK > 64 ? 128 : 64, L) <= 160 * 1024;
}
template <typename TIn>
hipError_t launch_f32_mma_typed(const F32Args& a, int S, int L, hipStream_t stream) {
    const int n = (a.DQK + 63) / 64;
    if (L == 16) {
        if (n == 1) return launch_f32_mma<TIn, 16, 1>(a, S, stream);
        if (n == 2) return launch_f32_mma<TIn, 16, 2>(a, S, stream);
        if (n <= 4) return launch_f32_mma<TIn, 16, 4>(a, S, stream);
        return launch_f32_mma<TIn, 16, 8>(a, S, stream);
    }
    if (L == 32) {
        if (n == 1) return launch_f32_mma<TIn, 32, 1>(a, S, stream);
        if (n == 2) return launch_f32_mma<TIn, 32, 2>(a, S, stream);
        return launch_f32_mma<TIn, 32, 4>(a, S, stream);
    }
    if (n == 1) return launch_f32_mma<TIn, 64, 1>(a, S, stream);
    return launch_f32_mma<TIn, 64, 2>(a, S, stream);
}

hipError_t launch_chunk_f32(mlstm_dtype dt, const ChunkArgs& a, hipStream_t stream) {
    const int S = a.B * a.NH;
    // a launch has at most 2^32 - 1 threads; past that (more than a million sequences) the VALU kernel's wider
    // dv tiles still fit
    const bool fits = static_cast<int64_t>(S) * (a.DV / 16) * (64 * kMmaW) < (int64_t(1) << 32);
    if (fits && f32_mma_supported(a.DQK, a.DV, a.L)) {
        const F32Args m{a.q, a.k, a.v, a.ipre, a.fpre, a.C0, a.n0, a.m0, a.T, a.DQK, a.DV, a.h, a.CT, a.nT, a.mT};
        return dt == MLSTM_BF16 ? launch_f32_mma_typed<bf16_t>(m, S, a.L, stream) : launch_f32_mma_typed<float>(m, S, a.L, stream);
    }
    const int dvt = chunk_f32_tile(a.DQK, a.DV, a.L);
    const size_t lds = f32_lds_floats(a.DQK, dvt, a.L) * sizeof(float);
    const dim3 grid(static_cast<unsigned>(a.B * a.NH * (a.DV / dvt)));
    if (dt == MLSTM_BF16) {
        hipLaunchKernelGGL(chunk_f32_kernel<bf16_t>, grid, dim3(kF32Threads), lds, stream,
                           static_cast<const bf16_t*>(a.q), static_cast<const bf16_t*>(a.k),
                           static_cast<const bf16_t*>(a.v), a.ipre, a.fpre, a.C0, a.n0, a.m0, a.T, a.DQK,
                           a.DV, a.L, dvt, static_cast<bf16_t*>(a.h), a.CT, a.nT, a.mT);
    } else {
        hipLaunchKernelGGL(chunk_f32_kernel<float>, grid, dim3(kF32Threads), lds, stream,
                           static_cast<const float*>(a.q), static_cast<const float*>(a.k),
                           static_cast<const float*>(a.v), a.ipre, a.fpre, a.C0, a.n0, a.m0, a.T, a.DQK,
                           a.DV, a.L, dvt, static_cast<float*>(a.h), a.CT, a.nT, a.mT);
    }
    return hipGetLastError();
}

#ifdef MLSTM_DEBUG
MLSTM_DEBUG_READER(debug_flags_chunk_f32)
#endif

}  // namespace mlstm

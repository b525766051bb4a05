// Device pieces shared by the chunkwise prefill kernel and the backward's chunk walk (bf16, the
// xLSTM 7B head shape): the workgroup shape, the chunk configuration, the per-chunk gate quantities
// and the gate phase that computes them, V staging with its transposition on the matrix cores, and
// the sequence addressing.  Everything lives in an anonymous namespace, so each translation unit that
// includes this header has its own copy.
#pragma once
#include <type_traits>

#include "mfma_common.h"

namespace mlstm {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = 8;
constexpr int kGateWave = kWaves - 1; // the wave with the least MFMA work runs the gate scans
constexpr float kRenorm = -20.0f;     // rescale C eagerly when its lazy log-scale would drop below this
constexpr float kRenormAlways = 1.0f; // a lazy log-scale is never positive

// Tokens per chunk; a call's own chunk length only shapes its segments (see launch_chunk_mfma).
constexpr int kL = 64;
struct Cfg {
    static constexpr int NDB = 2;                   // d blocks staged per chunk
    static constexpr int DB = kDQK / NDB;           // 128
    static constexpr int DT = DB / 16;              // 16-row C tiles per d block
    // row pitch (elements) of Q and K blocks: 288 bytes keep the 16-byte row reads of 16 consecutive rows
    // free of bank conflicts
    static constexpr int QP = DB + 16;
    static constexpr int SP = kL + 16;              // row pitch of S~ (160 bytes)
    static constexpr int QKE = kL * QP;             // elements of one Q or K block buffer
    // Wave split of the workgroup's 256 x 128 slice of C: DH d partitions x (8 / DH) column
    // groups of VT 16-column tiles.  Two partitions halve the Q and K^T operand reads of
    // (iii) and (iv) at the price of summing the two partial read-outs of (iii) through LDS.
    static constexpr int DH = 2;
    static constexpr int VT = 2;
    static constexpr int NVG = kWaves / DH;
    // V is kept in LDS transposed (rows v, tau contiguous, pitch TP), once plain for (ii) and once
    // scaled by the C-update key weights for (iv), so both read it with plain 16-byte row reads
    static constexpr int TP = kL + 8;
};

// Per-chunk gate quantities, written one chunk ahead by the gate wave.  kF32N: the n-update weights in fp32, for
// the backward, which branches on |q . n + ...| against the floor, so that n's rounding decides rows close to it.
template <bool kF32N>
struct alignas(16) GateBuf {
    float x2[kL];       // (i~ - b) * log2 e
    float M2[kL];       // M * log2 e (0 for a row with no input at all)
    int R[kL];          // last restart (forget gate exactly zero) at or before the row, -1: none
    float interC[kL];   // exp(m_prev - M + s) / sqrt(DQK): scale of C_acc^T Q^T
    float interN[kL];   // exp(m_prev - M) / sqrt(DQK):     scale of Q n
    float floorv[kL];   // exp(-(b + M))
    float wC[kL];       // C-update weights exp(x - M_L - s_new)
    std::conditional_t<kF32N, float[kL], uint16_t[2][kL]> wb;   // n-update weights exp(x - M_L): fp32, or bf16 hi / lo rows
    float scal[4];      // [0] n decay, [1] m_next, [2] s_new, [3] eager C scale (1: none)
};

struct VRegs {
    static constexpr int N = (kL * kDVT / 8) / kThreads;   // 16-byte pieces of a V chunk per thread
    u32x4_t v[N];
};

// V pieces in the MFMA A-operand layout for vt_transpose: piece i of wave w has lane (l16, g16) holding
// V[tau 16 a + l16][v 32 b + 8 g16 + 0..7], (a, b) = (w % 4, N (w / 4) + i); the workgroup's pieces cover
// the 64 x 128 chunk once, and a wave's pieces are neighbours in v, so that the two 64-byte halves of a
// memory line are requested one after the other.
__device__ __forceinline__ int v_piece_b(int wave, int i) { return VRegs::N * (wave >> 2) + i; }
__device__ __forceinline__ void load_v_tr(VRegs& r, const SeqRsrc& R, int t0, int v0, int wave, int lane, uint32_t rv) {
    static_assert(VRegs::N * kWaves == (kL / 16) * (kDVT / 32), "pieces of one 64 x 128 chunk");
    const uint32_t soff = v0 * 2;   // the row offset goes in the per-lane offset
    int ln = lane;   // opaque: the offsets are recomputed per call rather than held across the loop
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int i = 0; i < VRegs::N; ++i) {
        const int a = wave & 3, b = v_piece_b(wave, i);
        r.v[i] = bload128(R.v, static_cast<uint32_t>(t0 + 16 * a + (ln & 15)) * rv + (32 * b + 8 * (ln >> 4)) * 2, soff);
    }
}
using VtPacked = u32x2_t[2 * VRegs::N];
// The transposition on the matrix cores: D = A E_h with A a piece (16 tau x 32 v) and E_h the 32 x 16
// one-hot selection of its columns 16 h + 0..15 (exact in fp32).  Lane (n = l16, g16) of D holds
// V[tau 16 a + 4 g16 + j][v 32 b + 16 h + n], j = 0..3: four consecutive tau of one row of V^T, kept
// packed in pv until the stores below.
// One-hot selection E_h (32 x 16, columns 16 h + 0..15 of a 32-column piece) in the B-operand layout:
// lane (l16, g16) holds k slots 8 g16 + 0..7 of column l16, whose one (if any) is slot 16 h + l16.
// That slot lies in the lane's eight when 16 h + l16 - 8 g16 is in 0..7, i.e. when g16 = 2 h + l16 / 8,
// and is then slot l16 % 8 of them: register (l16 / 2) % 4, half l16 % 2.  Built from an opaque copy
// of the lane index so that it is not hoisted out of the chunk loop (eight more registers held
// across the loop would spill).
__device__ __forceinline__ void onehot_pair(u32x4_t (&E)[2], int lane) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int sel = (ln >> 1) & 3;
    const int gh = (ln >> 4) - ((ln >> 3) & 1);   // 2 h for the h whose column this lane can hold
    const uint32_t one = (ln & 1) ? 0x3F800000u : 0x3F80u;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const uint32_t oh = (gh == 2 * h) ? one : 0u;
#pragma unroll
        for (int d = 0; d < 4; ++d) E[h][d] = (sel == d) ? oh : 0u;
    }
}

__device__ __forceinline__ void vt_transpose(VtPacked& pv, const VRegs& r, int lane) {
    u32x4_t E[2];
    onehot_pair(E, lane);
#pragma unroll
    for (int i = 0; i < VRegs::N; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4_t d = mfma16(r.v[i], E[h], f32x4_t{});
            pv[2 * i + h] = u32x2_t{pack_bf16x2(d[0], d[1]), pack_bf16x2(d[2], d[3])};
        }
}

__device__ __forceinline__ void load_gates(float& gi, float& gf, const SeqRsrc& R, int t0, int lane) {
    const uint32_t goff = static_cast<uint32_t>(t0 + lane) * 4;   // range-checked: zero past the end
    gi = bloadf(R.ig, goff, 0);
    gf = bloadf(R.fg, goff, 0);
}


// Gate phase of one chunk (run by one wave): in-chunk prefix sums and maxima, the max
// state, the lazy C scale, and every per-row scale of the chunk.  m_prev and s_cur
// carry the max state and the lazy log-scale from chunk to chunk.  Rows at or beyond
// nvalid (the partial last chunk of a sequence) are neutral tokens: no input (x = -inf)
// and no decay (logsig f~ = 0), so they leave the state unchanged.
//
// A forget gate of exactly zero (f~ = -inf, a document border) restarts the state: nothing
// before that token reaches it or any later token.  The prefix sum b skips the restart token
// (the decay from s to t over tokens s+1..t never includes a restart for the pairs that
// survive), every row keeps R, its last restart at or before it, and the row's maxima, weights
// and entry-state terms cover only the tokens from R on.  A chunk that holds a restart drops
// its entry state: C and n are scaled by zero before this chunk's keys are added.
template <bool kF32N>
__device__ __forceinline__ void gate_phase(GateBuf<kF32N>& Gb, float gi, float gf, float& m_prev,
                                           float& s_cur, int lane, int nvalid, float renorm = kRenorm) {
    static_assert(kL == 64, "one token per lane");
    const bool ok = lane < nvalid;
    const float lg = ok ? flogsig(gf) : 0.0f;
    const bool rs = (lg == -INFINITY);
    // restarts are rare: a chunk without one (a wave-uniform test) takes the plain scans
    const bool any_restart = __builtin_amdgcn_ballot_w64(rs) != 0;
    const float b = wave_incl_sum(rs ? 0.0f : lg);
    const float x = ok ? gi - b : -INFINITY;
    float r = -1.f, p;
    if (any_restart) {
        r = wave_incl_max(rs ? static_cast<float>(lane) : -1.0f);
        p = wave_seg_incl_max(x, rs);
    } else {
        p = wave_incl_max(x);
    }
    const float pL = lane63(p);
    const float bL = lane63(b);
    const float rL = lane63(r);
    const bool restart = (rL >= 0.0f);
    const float ML = restart ? pL : fmaxf(m_prev, pL);
    // an empty state (m = -inf) has nothing to decay, and a restart drops the state
    const bool empty = restart || (m_prev == -INFINITY);
    const float dlog = empty ? 0.0f : m_prev - ML;
    const float s_try = s_cur + dlog;
    const bool eager = restart || s_try < renorm;
    const float s_new = eager ? 0.0f : s_try;
    auto emit = [&](int tau, float bb, float xx, float pp, float rr) {
        const bool fresh = (rr >= 0.0f);   // a restart at or before this row: no entry-state term
        const float M = fresh ? pp : fmaxf(m_prev, pp);
        Gb.x2[tau] = xx * kLog2e;
        Gb.M2[tau] = (M == -INFINITY) ? 0.0f : M * kLog2e;
        Gb.R[tau] = static_cast<int>(rr);
        Gb.interC[tau] = (fresh || M == -INFINITY) ? 0.0f : fexp(m_prev - M + s_cur) * kQScale;
        Gb.interN[tau] = (fresh || M == -INFINITY) ? 0.0f : fexp(m_prev - M) * kQScale;
        Gb.floorv[tau] = fexp(-(bb + M));
        const bool none = (xx == -INFINITY) || (static_cast<float>(tau) < rL);
        Gb.wC[tau] = none ? 0.0f : fexp(xx - ML - s_new);
        const float wn = none ? 0.0f : fexp(xx - ML);
        if constexpr (kF32N) {
            Gb.wb[tau] = wn;
        } else {
            const uint16_t whi = f32_to_bf16(wn);
            Gb.wb[0][tau] = whi;
            Gb.wb[1][tau] = f32_to_bf16(wn - bf16_to_f32(whi));
        }
    };
    emit(lane, b, x, p, r);
    const float m_next = bL + ML;
    if (lane == 0) {
        Gb.scal[0] = (empty || ML == -INFINITY) ? 0.0f : fexp(m_prev - ML);
        Gb.scal[1] = m_next;
        Gb.scal[2] = s_new;
        Gb.scal[3] = restart ? 0.0f : (eager ? fexp(s_try) : 1.0f);
    }
    m_prev = m_next;
    s_cur = s_new;
}

// First row of sequence s = (batch b, head s - b NH), written as s st_h + b (st_b - NH st_h) with
// st = {st_b - NH st_h, st_h}, and the byte span of its T rows of D elements.  b = floor(s / NH)
// comes from a multiply by the host's nh_magic (nh_magic = 0 stands for NH = 1, b = s): it is exact
// while s NH < 2^32 (the host checks this for strided calls), and contiguous rows have st[0] = 0.
// (An integer division, the form b st_b + (s - b NH) st_h, and this helper itself in the chunk
// kernel all made the compiler's code for its chunk loop markedly slower; the chunk kernel writes the
// same sum out in place.)
__device__ __forceinline__ const uint16_t* seq_rows(const uint16_t* p, int s, uint32_t nh_magic, const int64_t (&st)[2]) {
    const int b = nh_magic ? static_cast<int>(__umulhi(static_cast<uint32_t>(s), nh_magic)) : s;
    return p + static_cast<int64_t>(s) * st[1] + static_cast<int64_t>(b) * st[0];
}
__device__ __forceinline__ uint32_t seq_span(int T, uint32_t row_bytes, int D) {
    return T > 0 ? static_cast<uint32_t>(T - 1) * row_bytes + static_cast<uint32_t>(D) * 2u : 0u;
}

}  // namespace
}  // namespace mlstm

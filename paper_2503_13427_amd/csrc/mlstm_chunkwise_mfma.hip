// Chunkwise-parallel mLSTM forward on bf16 MFMA for the xLSTM 7B head shape
// (DQK = 256, DV = 512; Sec. 3.1 sets d_qk = d_hv / 2 and d_hv = 512), in chunks
// of 64 tokens.
//
// Math.  The chunkwise form of Sec. 2 ("Training Mode") with the sub-steps of
// App. D.1.  Per chunk, with the entry state (C, n, m_prev), in-chunk prefix
// sums b of logsig(f~), x = i~ - b, p_tau = max_{sig<=tau} x_sig and
// M_tau = max(m_prev, p_tau) (so the max state of Eq. 2 is m_tau = b_tau + M_tau):
//
//   S~^T[sig][tau] = (K Q^T)[sig][tau] / sqrt(DQK) * exp(x_sig - M_tau)   (sig <= tau, else 0)
//   N^T            = exp(m_prev - M_tau)/sqrt(DQK) * (C^T Q^T)  +  V^T S~^T
//   den_tau        = exp(m_prev - M_tau)/sqrt(DQK) * (Q n)_tau  +  rowsum_tau(S~)
//   h_tau          = N^T[:, tau] / max(|den_tau|, exp(-(b_tau + M_tau)))
//   C <- exp(m_prev - M_L) C + (w K)^T V,  n <- exp(m_prev - M_L) n + K^T w,
//   w_tau = exp(x_tau - M_L),  m_next = b_L + M_L.
// Every exponent is a difference against M and is <= 0 by construction.
//
// Lazily scaled matrix memory.  The accumulators hold C_acc with C = C_acc e^{s}.
// A chunk's decay is folded into s (s += m_prev - M_L) and into the key weights
// of the update (w e^{-s} <= e^{-kRenorm}), so the 64 accumulator registers of C in
// a wave are not rescaled by VALU work in most chunks; when s would fall below
// kRenorm the chunk applies the decay eagerly instead (C_acc *= e^{s + m_prev - M_L},
// between the read-out (iii) and the update (iv)) and s returns to 0.  The
// inter-chunk term uses exp(m_prev - M_tau + s); the exit state is C_acc e^{s}.
//
// Products and their MFMA mapping (gfx950 bf16 16x16x32 MFMA, fp32 accumulate):
//   (i)   S^T = K Q^T             A = K rows, B = Q rows (both d-contiguous)
//   (ii)  N^T += V^T S~^T         A = V^T rows, B = S~ rows
//   (iii) N^T += C^T Q^T          A = the C accumulators of (iv), converted to bf16 in
//                                 registers, B = Q rows
//   (iv)  C += K^T (w e^{-s} V)   A = K read transposed, B = (w e^{-s} V)^T rows
//   Q n and K^T w                 the fp32 normaliser and weights split into bf16 hi + lo
//                                 rows (relative error ~2^-17)
// "Read transposed" is the LDS transpose read of gfx950 (ds_read_b64_tr_b16): in each
// 16-lane group, lane 4s+q supplies 4 consecutive elements of row s of a 4 x 16 tile and
// lane c receives column c, so a row-major [k][m] tile arrives k-contiguous, as an MFMA
// operand wants it.  Q and K live in LDS in their natural layout.  V is transposed once per
// chunk on the matrix cores instead (a piece in the A-operand layout times a one-hot
// selection, exact) and kept in LDS as V^T and as the key-weighted (w e^{-s} V)^T, so (ii)
// and (iv) read it with plain 16-byte row reads.
// (iii) consumes C in the accumulator layout of (iv): the contraction index d is
// permuted consistently in both operands.  Outputs come out transposed (rows v,
// columns tau), so each lane stores runs of four consecutive v of one h row.
//
// Work decomposition.  One workgroup of 8 waves (two per SIMD, so one wave's
// LDS and memory waits are covered by the other's MFMAs) owns one (sequence,
// 128-column dv tile, segment) and walks the segment's chunks in order.  Each wave
// owns 64 accumulator registers of C for the whole segment (a 128 x 32 slice,
// one of two d partitions of a 32-column group); S~, Q n
// and the gates are computed once per workgroup.
// Q and K are staged in two d blocks of 128;
// the next block (and the next chunk's V and gates) is prefetched into registers
// while the current block is multiplied.  The four dv tiles of a (sequence,
// segment) are dispatched consecutively onto one XCD so their shared Q/K reads
// hit one L2.
//
// Segment-parallel schedule (optional workspace).  With G segments per sequence:
// (1) local_state_kernel computes the state of each of the first G-1 segments (split
// into R sub-segments of at most kLocMax tokens) from an empty state, as one weighted
// contraction over its tokens; (2) a combine kernel scans those local states into each
// segment's entry state, m_in' = max(gsum + m_in, m_loc),
// C_in' = e^{gsum + m_in - m_in'} C_in + e^{m_loc - m_in'} C_loc; (3) the chunkwise
// kernel runs every segment from its entry state.
#include <mutex>

#include "chunk_common.h"
#include "launch.h"

namespace mlstm {
namespace {

struct Smem {
    using C = Cfg;
    // d-block set s: Q [tau * QP + d], then K the same way; d block p uses set p % 2
    uint16_t QK[2][2 * C::QKE];
    // [0] V^T[v][tau] and [1] (w e^{-s} V)^T[v][tau] of the current chunk (this workgroup's 128 columns)
    uint16_t Vs[2][kDVT * C::TP];
    uint16_t St[kL * C::SP];                        // S~[tau][sig]
    uint16_t nb[2][2][kDQK];                       // normaliser as bf16 hi / lo rows, double-buffered
    float n[2][kDQK];                              // fp32 normaliser, double-buffered across chunks
    float dq[kL];                                   // Q n_{k-1} (unscaled q)
    float rs[kL * (kL / 16)];                        // row sums of S~ per (sigma block, tau)
    __device__ float& rsum_at(int tau, int sb) { return rs[sb * kL + tau]; }
    GateBuf<false> G[2];                               // by chunk parity
    // partial read-outs exchanged between the two d partitions of a column group (DH = 2):
    // [column group][v tile][tau tile][lane] as float4
    float X[C::NVG * C::VT * (kL / 16) * 64 * 4];
};
static_assert(sizeof(Smem) <= 160 * 1024, "LDS budget");

// Per-thread staging registers: one Q/K d block in flight (V: VRegs).
struct QKRegs {
    static constexpr int N = (kL * Cfg::DB / 8) / kThreads;   // 16-byte pieces per thread per matrix
    u32x4_t q[N];
    u32x4_t k[N];
};


// Q and K rows are 512 bytes, V rows 1024 bytes; offsets are in bytes.
// The chunk's row offset t0 rides in the per-lane offset with the row, so rows past the end of a
// sequence fall outside the buffer range and read as zero in a partial last chunk; the scalar offset
// carries only the column base.  Row strides (bytes) come from the call: q, k and v may be strided
// views of one projection output.
__device__ __forceinline__ void load_qk(QKRegs& r, const SeqRsrc& R, int t0, int p, int tid, uint32_t rq,
                                        uint32_t rk) {
    constexpr int DB = Cfg::DB, PR = DB / 8;   // 16-byte pieces per row
    const uint32_t soff = p * (DB * 2);
#pragma unroll
    for (int i = 0; i < QKRegs::N; ++i) {
        const int item = tid + i * kThreads;
        const uint32_t row = static_cast<uint32_t>(t0 + item / PR), col = 16 * (item % PR);
        r.q[i] = bload128(R.q, row * rq + col, soff);
        r.k[i] = bload128(R.k, row * rk + col, soff);
    }
}
__device__ __forceinline__ void store_qk(uint16_t* Qd, uint16_t* Kd, const QKRegs& r, int tid) {
    constexpr int PR = Cfg::DB / 8, QP = Cfg::QP;
#pragma unroll
    for (int i = 0; i < QKRegs::N; ++i) {
        const int item = tid + i * kThreads;
        const int off = (item / PR) * QP + 8 * (item % PR);
        MLSTM_CHECK(off >= 0 && off + 8 <= Cfg::QKE, kDbgChunkMfma);
        *reinterpret_cast<u32x4_t*>(&Qd[off]) = r.q[i];
        *reinterpret_cast<u32x4_t*>(&Kd[off]) = r.k[i];
    }
}
// (w V)^T from the packed V^T: row weights wC of the chunk, rounded to bf16 once
__device__ __forceinline__ void vt_store_scaled(uint16_t* VwT, const VtPacked& pv, const float* wC, int wave,
                                                int lane) {
    constexpr int TP = Cfg::TP;
    const int l16 = lane & 15, g16 = lane >> 4;
#pragma unroll
    for (int i = 0; i < VRegs::N; ++i) {
        const int a = wave & 3, b = v_piece_b(wave, i);
        const int tau = 16 * a + 4 * g16;
        const f32x4_t w = *reinterpret_cast<const f32x4_t*>(&wC[tau]);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const u32x2_t x = pv[2 * i + h];
            u32x2_t o;
            o[0] = pack_bf16x2(lo_f32(x[0]) * w[0], hi_f32(x[0]) * w[1]);
            o[1] = pack_bf16x2(lo_f32(x[1]) * w[2], hi_f32(x[1]) * w[3]);
            MLSTM_CHECK(32 * b + 16 * h + l16 < kDVT && tau + 4 <= TP, kDbgChunkMfma);
            *reinterpret_cast<u32x2_t*>(&VwT[(32 * b + 16 * h + l16) * TP + tau]) = o;
        }
    }
}
__device__ __forceinline__ void vt_store_plain(uint16_t* VtT, const VtPacked& pv, int wave, int lane) {
    constexpr int TP = Cfg::TP;
    const int l16 = lane & 15, g16 = lane >> 4;
#pragma unroll
    for (int i = 0; i < VRegs::N; ++i) {
        const int a = wave & 3, b = v_piece_b(wave, i);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            MLSTM_CHECK(32 * b + 16 * h + l16 < kDVT && 16 * a + 4 * g16 + 4 <= TP, kDbgChunkMfma);
            *reinterpret_cast<u32x2_t*>(&VtT[(32 * b + 16 * h + l16) * TP + 16 * a + 4 * g16]) = pv[2 * i + h];
        }
    }
}
struct ChunkKernelArgs {
    const uint16_t* q;
    const uint16_t* k;
    const uint16_t* v;
    const float* ipre;
    const float* fpre;
    const float* C0;   // entry state of segment 0 (NULL: zero state, m = 0)
    const float* n0;
    const float* m0;
    float* ws;         // segment slots (NULL when G == 1)
    int S;             // sequences (B NH)
    int T;
    int G;             // segments per sequence
    int R;             // local sub-segments per segment; segment g >= 1 enters from slot g R - 1
    int NS;            // local slots per sequence, (G - 1) R
    int seg_chunks;    // chunks per segment (last may be shorter)
    int eager_chunk;   // a chunk whose state is rescaled eagerly (see launch_chunk_mfma), or -1
    uint16_t* h;
    float* CT;
    float* nT;
    float* mT;
    uint32_t nh_magic;             // floor(2^32 / NH) + 1, or 0 for NH = 1 (see seq_rows)
    // element strides of q, k, v: [0] batch stride - NH head stride, [1] head stride (see seq_rows)
    int64_t sq[2], sk[2], sv[2];
    uint32_t rq, rk, rv;           // their row (token) strides in bytes
};


// row pitch (floats) of the entry-state staging of a 256 x 128 tile in LDS: 528 bytes puts the
// rows 8 apart that one read of the accumulator pickup touches in different banks
constexpr int kStageP = kDVT + 4;
static_assert(kDQK * kStageP * 4 <= sizeof(Smem), "staging");


// Staging order (one Q/K block and one V chunk in registers at a time): block 0 of a chunk is stored during
// the previous chunk (at the barrier that opens block 1), block 1 at the top of the chunk.  The next chunk's
// block p is requested after block p's logits, its V during block 0's read-out; V is transposed in registers
// at the barrier that opens block 1, its weighted copy goes to LDS after the S~ barrier (once this chunk's
// (iv) is done and the next chunk's weights are known), its plain copy at the top of the next chunk (once
// this chunk's (ii) is done).  The loads run in every chunk (the last one repeats its own): behind a
// branch the compiler cannot count the loads in flight and waits for all of them, and a harmless change of
// the code around has moved such a wait right behind the loads (950 instead of 795 us for 8 x 8192 tokens).
// What the loads feed is left out in the last chunk (with it, calls of one chunk took 13.4 instead of 13.0 us).
__global__ void __launch_bounds__(kThreads, 1) chunk_mfma_kernel(ChunkKernelArgs A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    Smem& S = *reinterpret_cast<Smem*>(smem_raw);
    using CF = Cfg;
    constexpr int QP = CF::QP, SP = CF::SP, NB = kL / 16, DB = CF::DB, DT = CF::DT, NDB = CF::NDB;
    constexpr int NT_S = NB * (NB + 1) / 2;          // causal 16x16 tiles of S^T
    constexpr int MAXT = (NT_S + kWaves - 1) / kWaves;
    constexpr int NTT = kL / 16;                       // 16-wide tau tiles
    constexpr int NKS = kL / 32;                       // k steps of 32 along the chunk
    constexpr int NUT = (DB / 16 + kWaves - 1) / kWaves;   // 16-col n-update tiles per wave per block

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g16 = lane >> 4;  // k group of the 16x16x32 operands, also the transpose-read group
    const int l16 = lane & 15;
    constexpr int DH = CF::DH, VT = CF::VT, NVG = CF::NVG;
    constexpr int NQ = DT / DH;                 // this wave's 16-row C tiles per d block
    const int vg = wave % NVG;                  // column group
    const int dh = wave / NVG;                  // d partition: tiles dt = q DH + dh of every d block
    auto vcol = [&](int vt) { return 16 * (vg * VT + vt); };   // first column of v tile vt
    // d row of element j of accumulator tile t (see the entry state)
    auto cdrow = [&](int t, int j) {
        const int q = t % NQ;
        return (t / NQ) * DB + 32 * ((q / 2) * DH + dh) + 8 * g16 + 4 * (q % 2) + j;
    };
    const bool gate_wave = (wave == kGateWave);
    // Q n tile of this wave (>= NTT: none): the waves after the two that hold two S tiles take it
    const int dqt = wave - 2;
    const bool dq_wave = (dqt >= 0 && dqt < NTT);

    const int wi = work_index();
    const int tile = wi % kNTile;
    const int sg = wi / kNTile;
    const int g = sg % A.G;
    const int s = sg / A.G;
    const int v0 = tile * kDVT;
    const int nc_total = (A.T + kL - 1) / kL;   // the last chunk may be partial
    const int c_begin = g * A.seg_chunks;
    const int c_end = min(nc_total, c_begin + A.seg_chunks);

    SeqRsrc P;
    // the sequence's rows, written out here rather than through seq_rows: this form keeps the
    // compiler's code for the chunk loop as fast as with contiguous-only addressing
    const int bq = A.nh_magic ? static_cast<int>(__umulhi(static_cast<uint32_t>(s), A.nh_magic)) : s;
    P.q = make_rsrc(A.q + static_cast<int64_t>(s) * A.sq[1] + static_cast<int64_t>(bq) * A.sq[0], seq_span(A.T, A.rq, kDQK));
    P.k = make_rsrc(A.k + static_cast<int64_t>(s) * A.sk[1] + static_cast<int64_t>(bq) * A.sk[0], seq_span(A.T, A.rk, kDQK));
    P.v = make_rsrc(A.v + static_cast<int64_t>(s) * A.sv[1] + static_cast<int64_t>(bq) * A.sv[0], seq_span(A.T, A.rv, kDV));
    P.ig = make_rsrc(A.ipre + static_cast<int64_t>(s) * A.T, static_cast<uint32_t>(A.T) * 4);
    P.fg = make_rsrc(A.fpre + static_cast<int64_t>(s) * A.T, static_cast<uint32_t>(A.T) * 4);
    P.h = make_rsrc(A.h + static_cast<int64_t>(s) * A.T * kDV, static_cast<uint32_t>(A.T) * kDV * 2);

    // ---- entry state ------------------------------------------------------------------------
    // C tiles come in pairs over 32 consecutive d: in pair pp of a d block, tile e (0, 1) holds the d
    // with (d mod 8) / 4 == e.  This wave owns pairs pp = pq DH + dh; Cacc[p NQ + 2 pq + e][vt] lane
    // holds C[p DB + 32 pp + 8 g16 + 4 e + j][vcol(vt) + l16], j = 0..3, so the read-out (iii) finds
    // the 8 d of its k slots contiguous in Q.
    f32x4_t Cacc[NDB * NQ][VT];
    const float* Cin = nullptr;
    const float* nin = nullptr;
    float m_prev;
    if (g == 0) {
        Cin = A.C0 ? A.C0 + static_cast<int64_t>(s) * kDQK * kDV : nullptr;
        nin = A.n0 ? A.n0 + static_cast<int64_t>(s) * kDQK : nullptr;
        m_prev = A.m0 ? A.m0[s] : 0.0f;
    } else {
        MLSTM_CHECK(s < A.S && g * A.R - 1 >= 0 && g * A.R - 1 < A.NS, kDbgChunkMfma);
        const float* slot = A.ws + (static_cast<int64_t>(s) * A.NS + g * A.R - 1) * kSlotFloats;
        Cin = slot;
        nin = slot + kDQK * kDV;
        m_prev = slot[kDQK * kDV + kDQK + 2];
    }
    MLSTM_CHECK(s < A.S, kDbgChunkMfma);
    // a segment entry slot is loaded after the first chunk's staging loads, so that their waits do not
    // include it
    const bool slot_entry = (Cin && g > 0);
    if (Cin && !slot_entry) {
        // C0: the workgroup's 256 x 128 tile in coalesced 16-byte pieces, staged in LDS (rows of
        // kStageP floats, before the chunk loop uses it) and picked up in the accumulator layout
        float* stage = reinterpret_cast<float*>(smem_raw);
#pragma unroll 4
        for (int i = 0; i < (kDQK * kDVT / 4) / kThreads; ++i) {
            const int f = tid + kThreads * i;
            const int row = f / (kDVT / 4), c4 = f % (kDVT / 4);
            *reinterpret_cast<f32x4_t*>(&stage[row * kStageP + 4 * c4]) =
                *reinterpret_cast<const f32x4_t*>(Cin + static_cast<int64_t>(row) * kDV + v0 + 4 * c4);
        }
        __syncthreads();
#pragma unroll
        for (int t = 0; t < NDB * NQ; ++t)
#pragma unroll
            for (int vt = 0; vt < VT; ++vt)
#pragma unroll
                for (int j = 0; j < 4; ++j) Cacc[t][vt][j] = stage[cdrow(t, j) * kStageP + vcol(vt) + l16];
        __syncthreads();   // the staging area is the LDS of the chunk loop
    } else if (!slot_entry) {
#pragma unroll
        for (int t = 0; t < NDB * NQ; ++t)
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) Cacc[t][vt] = f32x4_t{};
    }
    if (tid < kDQK) {
        const float nv = nin ? nin[tid] : 0.0f;
        S.n[0][tid] = nv;
        const uint16_t hi = f32_to_bf16(nv);
        S.nb[0][0][tid] = hi;
        S.nb[0][1][tid] = f32_to_bf16(nv - bf16_to_f32(hi));
    }
    float s_off = 0.0f;   // C = C_acc * e^{s_off}

    // gate wave state: max state and lazy scale after the last chunk whose gates it computed
    float g_m = m_prev, g_s = 0.0f;
    float gi = 0.f, gf = 0.f;

    QKRegs rqk;
    VRegs rv;
    VtPacked pv;   // the next chunk's V^T, packed, until its stores
    if (c_begin < c_end) {
        const int t0 = c_begin * kL;
        load_qk(rqk, P, t0, 0, tid, A.rq, A.rk);
        if (gate_wave) {
            load_gates(gi, gf, P, t0, lane);
            gate_phase(S.G[c_begin & 1], gi, gf, g_m, g_s, lane, A.T - t0, c_begin == A.eager_chunk ? kRenormAlways : kRenorm);
        }
        store_qk(S.QK[0], S.QK[0] + CF::QKE, rqk, tid);
        load_v_tr(rv, P, t0, v0, wave, lane, A.rv);
        vt_transpose(pv, rv, lane);
        __syncthreads();   // the first chunk's gates are visible
        vt_store_scaled(S.Vs[1], pv, S.G[c_begin & 1].wC, wave, lane);
        vt_store_plain(S.Vs[0], pv, wave, lane);
        load_qk(rqk, P, t0, 1, tid, A.rq, A.rk);
    }
    if (slot_entry) {
        // a segment entry slot (four rows interleaved): each accumulator tile is one 16-byte load
#pragma unroll
        for (int t = 0; t < NDB * NQ; ++t)
#pragma unroll
            for (int vt = 0; vt < VT; ++vt)
                Cacc[t][vt] = *reinterpret_cast<const f32x4_t*>(Cin + slot_c4(cdrow(t, 0) / 4, v0 + vcol(vt) + l16));
    }

    f32x4_t Nacc[VT][NTT];
    f32x4_t Sacc[MAXT];
    f32x4_t dqacc;

    for (int c = c_begin; c < c_end; ++c) {
        // transpose-read lane roles inside a 16-lane group (16x16x32 operands)
        const int tr_row = (l16 >> 2) + 8 * g16;   // + 4r + k base
        const int tr_col = 4 * (l16 & 3);           // + m/n base
        const int t0 = c * kL;
        const int cur = (c - c_begin) & 1;
        const int par = c & 1;
        const GateBuf<false>& Gc = S.G[par];
        __syncthreads();   // the previous chunk is done; block 0, V and the gates of this chunk are visible
        // block 1 -> set 1 (its readers in the previous chunk, the last d block and S~, are done)
        store_qk(S.QK[1], S.QK[1] + CF::QKE, rqk, tid);
        const int tn = min(c + 1, c_end - 1) * kL;   // the next chunk
        load_gates(gi, gf, P, tn, lane);
        // this chunk's plain V^T (its readers in the previous chunk are done); the next chunk's V
        if (c > c_begin) vt_store_plain(S.Vs[0], pv, wave, lane);
        const float decay_n = Gc.scal[0];
        const float m_next = Gc.scal[1];
        const float s_new = Gc.scal[2];
        const float c_scale = Gc.scal[3];   // != 1: apply this chunk's decay to C_acc eagerly
        const float* n_old = S.n[cur];
        float* n_new = S.n[cur ^ 1];
        const uint16_t* VtT = S.Vs[0];
        const uint16_t* VwT = S.Vs[1];

#pragma unroll
        for (int vt = 0; vt < VT; ++vt)
#pragma unroll
            for (int T = 0; T < NTT; ++T) Nacc[vt][T] = f32x4_t{};
#pragma unroll
        for (int i = 0; i < MAXT; ++i) Sacc[i] = f32x4_t{};
        dqacc = f32x4_t{};

#pragma unroll
        for (int p = 0; p < NDB; ++p) {
            const uint16_t* Qs = S.QK[p & 1];
            const uint16_t* Ks = S.QK[p & 1] + CF::QKE;
            if (p > 0) {
                __syncthreads();   // block p visible, block p - 1 fully read
                // block 0 of the next chunk; its V, transposed in registers
                if (c + 1 < c_end) {
                    store_qk(S.QK[0], S.QK[0] + CF::QKE, rqk, tid);
                    vt_transpose(pv, rv, lane);
                }
            }
            // (i) S^T += K_p Q_p^T on this wave's causal tiles
#pragma unroll
            for (int i = 0; i < MAXT; ++i) {
                const int t = wave + kWaves * i;
                if (t < NT_S) {
                    int tb = 0, rem = t;
                    while (rem > tb) { rem -= tb + 1; ++tb; }
                    const int sb = rem;
                    const uint16_t* qb = &Qs[(16 * tb + l16) * QP + 8 * g16];
                    const uint16_t* ka = &Ks[(16 * sb + l16) * QP + 8 * g16];
#pragma unroll
                    for (int ks = 0; ks < DB / 32; ++ks)
                        Sacc[i] = mfma16(*reinterpret_cast<const u32x4_t*>(ka + 32 * ks),
                                         *reinterpret_cast<const u32x4_t*>(qb + 32 * ks), Sacc[i]);
                }
            }
            load_qk(rqk, P, tn, p, tid, A.rq, A.rk);   // the next chunk's block p
            // Q n_{k-1} over this d block: A = Q rows, B = n as bf16 hi / lo columns
            if (dq_wave) {
                const uint16_t* qa = &Qs[(16 * dqt + l16) * QP + 8 * g16];
                const uint16_t* nbp = &S.nb[cur][l16 & 1][p * DB + 8 * g16];
#pragma unroll
                for (int ks = 0; ks < DB / 32; ++ks) {
                    const u32x4_t nbv = (l16 < 2) ? *reinterpret_cast<const u32x4_t*>(nbp + 32 * ks)
                                                  : u32x4_t{0u, 0u, 0u, 0u};
                    dqacc = mfma16(*reinterpret_cast<const u32x4_t*>(qa + 32 * ks), nbv, dqacc);
                }
            }
            // (iii) N^T += C_p^T Q_p^T over this wave's tile pairs: A from the two C tiles of a
            // pair (rows 4 g16 + j of each), converted to bf16 in registers, is k slot 8 g16 + i
            // = d 32 pp + 8 g16 + i; B = 16 bytes of a Q row, shared by the VT column tiles.
            // C goes in as a bf16 pair hi + lo (lo = C - hi, rounded again), so the read-out sees C
            // to about 2^-16: a single bf16 rounding of the state (2^-9) is what a row whose
            // read-out cancels (|C^T q| much smaller than the terms it sums) would amplify
#pragma unroll
            for (int pt = 0; pt < NQ / 2; ++pt) {
                const int q0 = p * NQ + 2 * pt;
                u32x4_t a[VT], alo[VT];
#pragma unroll
                for (int vt = 0; vt < VT; ++vt) {
                    const f32x4_t& c0 = Cacc[q0][vt];
                    const f32x4_t& c1 = Cacc[q0 + 1][vt];
                    a[vt][0] = pack_bf16x2(c0[0], c0[1]);
                    a[vt][1] = pack_bf16x2(c0[2], c0[3]);
                    a[vt][2] = pack_bf16x2(c1[0], c1[1]);
                    a[vt][3] = pack_bf16x2(c1[2], c1[3]);
                    alo[vt][0] = pack_bf16x2(c0[0] - lo_f32(a[vt][0]), c0[1] - hi_f32(a[vt][0]));
                    alo[vt][1] = pack_bf16x2(c0[2] - lo_f32(a[vt][1]), c0[3] - hi_f32(a[vt][1]));
                    alo[vt][2] = pack_bf16x2(c1[0] - lo_f32(a[vt][2]), c1[1] - hi_f32(a[vt][2]));
                    alo[vt][3] = pack_bf16x2(c1[2] - lo_f32(a[vt][3]), c1[3] - hi_f32(a[vt][3]));
                }
                const int dq0 = 32 * (pt * DH + dh) + 8 * g16;   // within the block
                if (p == 0 && pt == 0) load_v_tr(rv, P, tn, v0, wave, lane, A.rv);
                // the Q operand of the next tau tile is requested before this one's MFMAs are issued
                // (the scheduling fence keeps the compiler from waiting on each read in turn)
                u32x4_t b = *reinterpret_cast<const u32x4_t*>(&Qs[l16 * QP + dq0]);
#pragma unroll
                for (int T = 0; T < NTT; ++T) {
                    u32x4_t bn = b;
                    if (T + 1 < NTT) bn = *reinterpret_cast<const u32x4_t*>(&Qs[(16 * (T + 1) + l16) * QP + dq0]);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int vt = 0; vt < VT; ++vt) {
                        Nacc[vt][T] = mfma16(a[vt], b, Nacc[vt][T]);
                        Nacc[vt][T] = mfma16(alo[vt], b, Nacc[vt][T]);
                    }
                    b = bn;
                }
            }

            // (iv) C_p += K_p^T (w e^{-s} V): A = K read transposed (this wave's d tiles),
            // B = V read transposed and scaled by the C-update key weights in registers (rebuilt
            // per d block: a short live range is worth the extra transposed reads)
            if (c_scale != 1.0f) {
#pragma unroll
                for (int q = 0; q < NQ; ++q)
#pragma unroll
                    for (int vt = 0; vt < VT; ++vt) Cacc[p * NQ + q][vt] *= c_scale;
            }
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) {
                // the K^T operands first: their reads are in flight while the weighted V operand is
                // built (the fence keeps the compiler from sinking them below that VALU work)
                u32x4_t a[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) {
                    // tile (pair q / 2, half q % 2): columns 32 pp + 8 (l16 & 3) + 4 (q % 2) + 0..3
                    const uint16_t* kb = &Ks[(32 * ks + tr_row) * QP + 32 * ((q / 2) * DH + dh) + 2 * tr_col + 4 * (q % 2)];
                    a[q] = cat(tr_read(kb), tr_read(kb + 4 * QP));
                }
                __builtin_amdgcn_sched_barrier(0);
                // lane (n = column vcol(vt) + l16, k group g16) holds tau = 32 ks + 8 g16 + 0..7
                u32x4_t Vw[VT];
#pragma unroll
                for (int vt = 0; vt < VT; ++vt)
                    Vw[vt] = *reinterpret_cast<const u32x4_t*>(&VwT[(vcol(vt) + l16) * CF::TP + 32 * ks + 8 * g16]);
#pragma unroll
                for (int q = 0; q < NQ; ++q)
#pragma unroll
                    for (int vt = 0; vt < VT; ++vt)
                        Cacc[p * NQ + q][vt] = mfma16(a[q], Vw[vt], Cacc[p * NQ + q][vt]);
            }
            // n_p = decay n_p + K_p^T w: A = w as bf16 hi / lo rows, B = K read transposed
#pragma unroll
            for (int j = 0; j < NUT; ++j) {
                const int ut = wave * NUT + j;   // 16-column tile of this d block
                if (ut >= DB / 16) break;
                f32x4_t nacc = f32x4_t{};
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) {
                    const u32x4_t wa = (l16 < 2) ? *reinterpret_cast<const u32x4_t*>(&Gc.wb[l16 & 1][32 * ks + 8 * g16])
                                                 : u32x4_t{0u, 0u, 0u, 0u};
                    const uint16_t* kb = &Ks[(32 * ks + tr_row) * QP + 16 * ut + tr_col];
                    const u32x4_t kt = cat(tr_read(kb), tr_read(kb + 4 * QP));
                    nacc = mfma16(wa, kt, nacc);
                }
                // rows 0 and 1 (hi and lo weights) of column l16 sit in lanes 0..15
                if (g16 == 0) {
                    const int d = p * DB + 16 * ut + l16;
                    const float nv = decay_n * n_old[d] + nacc[0] + nacc[1];
                    n_new[d] = nv;
                    const uint16_t hi = f32_to_bf16(nv);
                    S.nb[cur ^ 1][0][d] = hi;
                    S.nb[cur ^ 1][1][d] = f32_to_bf16(nv - bf16_to_f32(hi));
                }
            }
        }

        // gates of the next chunk, one chunk ahead; the other waves wait for them at the next
        // barrier, so the gate wave issues ahead of its SIMD partner meanwhile
        if (gate_wave && c + 1 < c_end) {
            __builtin_amdgcn_s_setprio(1);
            gate_phase(S.G[par ^ 1], gi, gf, g_m, g_s, lane, A.T - (t0 + kL), c + 1 == A.eager_chunk ? kRenormAlways : kRenorm);
            __builtin_amdgcn_s_setprio(0);
        }

        // finish Q n: columns 0 and 1 of the 16x16 tile are lanes l16 = 0 and 1
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float other = __shfl_down(dqacc[j], 1, 64);
            if (dq_wave && l16 == 0) S.dq[16 * dqt + 4 * g16 + j] = dqacc[j] + other;
        }
        // hand over the partial read-out of the tau tiles the other d partition finishes
        {
#pragma unroll
            for (int vt = 0; vt < VT; ++vt)
#pragma unroll
                for (int T = 0; T < NTT; ++T)
                    if ((T & 1) != dh) {
                        MLSTM_CHECK(((((vg * VT + vt) * NTT + T) * 64 + lane) * 4 + 4) <= static_cast<int>(sizeof(S.X) / 4),
                                    kDbgChunkMfma);
                        *reinterpret_cast<f32x4_t*>(&S.X[(((vg * VT + vt) * NTT + T) * 64 + lane) * 4]) = Nacc[vt][T];
                    }
        }
        // gate matrix on the S^T tiles -> S~ (bf16, tau-major) and row sums (fp32, before the
        // bf16 rounding); branch-free, one 16-byte read of the four sigma exponents per lane
#pragma unroll
        for (int i = 0; i < MAXT; ++i) {
            const int t = wave + kWaves * i;
            if (t < NT_S) {
                int tb = 0, rem = t;
                while (rem > tb) { rem -= tb + 1; ++tb; }
                const int sb = rem;
                const int tau = 16 * tb + l16;
                const float Mt = Gc.M2[tau];
                const int Rt = Gc.R[tau];
                const f32x4_t xs = *reinterpret_cast<const f32x4_t*>(&Gc.x2[16 * sb + 4 * g16]);
                float vals[4];
                float rsum = 0.f;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int sig = 16 * sb + 4 * g16 + j;
                    const float val = Sacc[i][j] * kQScale * fast_exp2(xs[j] - Mt);
                    // Rt <= sig <= tau as one unsigned comparison (Rt <= tau always)
                    vals[j] = (static_cast<unsigned>(sig - Rt) <= static_cast<unsigned>(tau - Rt)) ? val : 0.f;
                    rsum += vals[j];
                }
                u32x2_t o;
                o[0] = pack_bf16x2(vals[0], vals[1]);
                o[1] = pack_bf16x2(vals[2], vals[3]);
                MLSTM_CHECK(tau < kL && 16 * sb + 4 * g16 + 4 <= SP &&
                                tau * SP + 16 * sb + 4 * g16 + 4 <= kL * SP,
                            kDbgChunkMfma);
                *reinterpret_cast<u32x2_t*>(&S.St[tau * SP + 16 * sb + 4 * g16]) = o;
                rsum = sum_rows4(rsum);
                if (g16 == 0) S.rsum_at(tau, sb) = rsum;
            }
        }
        // zero the masked 16x16 tiles (sigma block T+1, tau block T) for even T: the k steps
        // of (ii) are 32 wide
        for (int T = 2 * wave; T < NTT; T += 2 * kWaves) {
            const int tau = 16 * T + l16;
            *reinterpret_cast<u32x2_t*>(&S.St[tau * SP + 16 * T + 16 + 4 * g16]) = u32x2_t{0u, 0u};
        }
        __syncthreads();
        // the next chunk's scaled V^T (its readers, (iv) of this chunk, are done; the next chunk's
        // weights are visible)
        if (c + 1 < c_end) vt_store_scaled(S.Vs[1], pv, S.G[par ^ 1].wC, wave, lane);
        // (ii) N^T = interC * N^T + V^T S~^T, then h = N^T / max(|den|, floor); each
        // d partition finishes the tau tiles T with T % 2 == dh, after adding the other's partial
#pragma unroll
        for (int T = 0; T < NTT; ++T) {
            if ((T & 1) != dh) continue;
            const int tau = 16 * T + l16;
            float den = Gc.interN[tau] * S.dq[tau];
#pragma unroll
            for (int sb = 0; sb <= T; ++sb) den += S.rsum_at(tau, sb);   // of sigma blocks 0..T
            const float hv = __builtin_amdgcn_rcpf(fmaxf(fabsf(den), Gc.floorv[tau]));
            const float ic = Gc.interC[tau];
#pragma unroll
            for (int vt = 0; vt < VT; ++vt) {
                f32x4_t acc = Nacc[vt][T];
                acc += *reinterpret_cast<const f32x4_t*>(&S.X[(((vg * VT + vt) * NTT + T) * 64 + lane) * 4]);
                acc *= ic;
#pragma unroll
                for (int ks = 0; ks <= T / 2; ++ks) {
                    MLSTM_CHECK(32 * ks + 8 * g16 + 8 <= SP && vcol(vt) + l16 < kDVT && 32 * ks + 8 * g16 + 8 <= CF::TP,
                                kDbgChunkMfma);
                    const u32x4_t b = *reinterpret_cast<const u32x4_t*>(&S.St[tau * SP + 32 * ks + 8 * g16]);
                    const u32x4_t va = *reinterpret_cast<const u32x4_t*>(&VtT[(vcol(vt) + l16) * CF::TP + 32 * ks + 8 * g16]);
                    acc = mfma16(va, b, acc);
                }
                u32x2_t o;
                o[0] = pack_bf16x2(acc[0] * hv, acc[1] * hv);
                o[1] = pack_bf16x2(acc[2] * hv, acc[3] * hv);
                // rows beyond T (a partial last chunk) fall outside the buffer range and are dropped
                __builtin_amdgcn_raw_buffer_store_b64(o, P.h,
                                                      static_cast<uint32_t>((t0 + tau) * kDV + v0 + vcol(vt) + 4 * g16) * 2, 0, 0);
            }
        }
        s_off = s_new;
        m_prev = m_next;
    }
    __syncthreads();

    // ---- exit state ---------------------------------------------------------------------------
    const int nfinal = (c_end - c_begin) & 1;
    float* Cout;
    float* nout;
    float* mout;
    const bool write_nm = (tile == 0);
    if (g != A.G - 1) return;
    Cout = A.CT + static_cast<int64_t>(s) * kDQK * kDV;
    nout = A.nT + static_cast<int64_t>(s) * kDQK;
    mout = A.mT + s;
    const float esc = expf(s_off);
#pragma unroll
    for (int t = 0; t < NDB * NQ; ++t) {
#pragma unroll
        for (int vt = 0; vt < VT; ++vt) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int d = cdrow(t, j);
                Cout[static_cast<int64_t>(d) * kDV + v0 + vcol(vt) + l16] = Cacc[t][vt][j] * esc;
            }
        }
    }
    if (write_nm && tid < kDQK) {
        nout[tid] = S.n[nfinal][tid];
        if (tid == 0) mout[0] = m_prev;
    }
}

// ---- local segment states as one weighted contraction ------------------------------------------
//
// From an empty state (C = 0, n = 0, m = -inf) the recurrence of Eq. 2-4 over tokens 1..N unrolls to
// a closed form: with b_t the prefix sums of logsig(f~_t) and x_t = i~_t - b_t,
//   m_N = b_N + X,  X = max_t x_t,   C_N = sum_t w_t k_t v_t^T,  n_N = sum_t w_t k_t,  w_t = exp(x_t - X)
// (every weight is <= 1).  With restarts (f~ = -inf) the prefix sums skip the restart tokens, only
// the tokens from the last restart R on carry weight (X is their maximum), and the sub-segment's
// logsig sum is -inf, so the combine drops whatever state entered it.
// A (sub-)segment's local state is therefore one contraction over its
// tokens, with no chunk recurrence: the gates are scanned once over the whole sub-segment, then
// 64-token tiles of K^T and V^T stream through LDS into the MFMA accumulators.  C and n are the
// same quantities the chunkwise update accumulates (bf16 w V operand, bf16 hi / lo weights for n).
constexpr int kLocTile = 64;                  // tokens per tile
constexpr int kLocMax = 4096;                 // tokens per sub-segment (weights held in LDS)
constexpr int kLocP = kLocTile + 8;           // K^T / V^T row pitch: 144 bytes

template <int NW>                             // bf16 rows of the n weights
struct LocSmem {
    uint16_t Kt[2][kDQK * kLocP];             // K^T[d][tau] of a tile, double-buffered
    uint16_t Vt[2][kDVT * kLocP];             // V^T[v][tau] (this workgroup's 128 columns)
    float w[kLocMax];                         // x_t, then the weights w_t
    uint16_t wb[NW][kLocMax];                 // the n weights as bf16 parts (hi, lo[, third])
    float red[3][kWaves];                     // per-wave scan totals, maxima, last restarts
};
static_assert(sizeof(LocSmem<3>) <= 160 * 1024, "LDS budget");

__device__ __forceinline__ uint32_t bload32(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
    return static_cast<uint32_t>(__builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}
// Column item regrouping: r[j] holds columns (c, c + 1) of row j as a bf16 pair; c0 / c1 receive
// column c / c + 1 over rows 0..7, in row order.
__device__ __forceinline__ void regroup(const uint32_t (&r)[8], u32x4_t& c0, u32x4_t& c1) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        c0[i] = __builtin_amdgcn_perm(r[2 * i + 1], r[2 * i], 0x05040100u);   // low halves
        c1[i] = __builtin_amdgcn_perm(r[2 * i + 1], r[2 * i], 0x07060302u);   // high halves
    }
}
// One tile in flight: two K column items (2 d x 8 tau) and one V column item (2 v x 8 tau) per
// thread, each read as eight 4-byte loads so the store side can write whole transposed rows.
struct LocRegs {
    uint32_t k[2][8];
    uint32_t v[8];
};
// kRagged: the tile may reach past the end of the sequence.  The range check of a buffer load covers the
// per-lane offset only, so the row goes there: row >= T gives an offset >= T row_bytes, which is past the
// buffer's last byte (seq_span <= T row_bytes), and reads as zero.  Tiles that are known to be full carry the
// row in the scalar offset (no address arithmetic per lane).
template <bool kRagged>
__device__ __forceinline__ void loc_load(LocRegs& r, const SeqRsrc& R, int t, int v0, int tid, uint32_t rk,
                                         uint32_t rv) {
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int item = tid + it * kThreads;
        const uint32_t row = 8 * (item / (kDQK / 2)), col = 4 * (item % (kDQK / 2));
#pragma unroll
        for (int j = 0; j < 8; ++j)
            r.k[it][j] = kRagged ? bload32(R.k, (row + t + j) * rk + col, 0)
                                 : bload32(R.k, row * rk + col, static_cast<uint32_t>(t + j) * rk);
    }
    const uint32_t row = 8 * (tid / (kDVT / 2)), col = 4 * (tid % (kDVT / 2));
#pragma unroll
    for (int j = 0; j < 8; ++j)
        r.v[j] = kRagged ? bload32(R.v, (row + t + j) * rv + col, v0 * 2)
                         : bload32(R.v, row * rv + col, static_cast<uint32_t>(t + j) * rv + v0 * 2);
}
__device__ __forceinline__ void loc_store(uint16_t* Kt, uint16_t* Vt, const LocRegs& r, int tid) {
    u32x4_t c0, c1;
#pragma unroll
    for (int it = 0; it < 2; ++it) {
        const int item = tid + it * kThreads;
        regroup(r.k[it], c0, c1);
        uint16_t* dst = &Kt[(2 * (item % (kDQK / 2))) * kLocP + 8 * (item / (kDQK / 2))];
        *reinterpret_cast<u32x4_t*>(dst) = c0;
        *reinterpret_cast<u32x4_t*>(dst + kLocP) = c1;
    }
    regroup(r.v, c0, c1);
    uint16_t* dst = &Vt[(2 * (tid % (kDVT / 2))) * kLocP + 8 * (tid / (kDVT / 2))];
    *reinterpret_cast<u32x4_t*>(dst) = c0;
    *reinterpret_cast<u32x4_t*>(dst + kLocP) = c1;
}

struct LocalArgs {
    const uint16_t* k;
    const uint16_t* v;
    uint32_t nh_magic;      // as in ChunkKernelArgs
    int64_t sk[2], sv[2];   // as in ChunkKernelArgs
    uint32_t rk, rv;        // their row strides in bytes
    const float* ipre;
    const float* fpre;
    float* ws;
    int S;             // sequences (B NH)
    int T;
    int NS;            // local slots per sequence: (G - 1) segments x R sub-segments
    int R;             // sub-segments per segment
    int seg_tokens;    // tokens per local segment (a multiple of kLocTile)
    // the reverse pass (kRev): per-token weights of the C and n parts, chunk decays, chunks per sequence
    const float* gd;
    const float* gw;
    const float* decay;
    int NC;
};
enum LocalMode { kFwd, kFwdHiLo, kRev };
// bf16 parts of the n weights: two (17 bits) for the prefill; three, all 24 bits, for the backward, whose branch
// |D| > floor reads n
template <LocalMode kMode>
constexpr int kLocalParts = kMode == kFwd ? 2 : 3;

// One workgroup per (sequence, local segment, sub-segment, dv tile); its slot receives C[:, tile],
// and (dv tile 0) n, m_loc and the segment's logsig sum.  kFwdHiLo: the weighted values w v enter the
// matrix cores as bf16 hi + lo (twice the products; the state to about 2^-17 instead of the 2^-9
// of one rounding per term), for the backward pass, whose gradients can cancel against the state.
// kRev: the same contraction for the backward's state gradients, over q and dh (in the places of k and v)
// of the segments 1..G-1: the weights come from memory, times the decays of the chunks before the token's
// in the sub-segment, and the slot ends with the product of all its decays.
// (the LDS footprint allows one workgroup per CU, two waves per SIMD: registers are not worth
// saving for a higher occupancy)
template <LocalMode kMode>
__global__ void __launch_bounds__(kThreads, 1) __attribute__((amdgpu_waves_per_eu(2, 2)))
local_state_kernel(LocalArgs A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    constexpr bool kHiLo = (kMode == kFwdHiLo);
    constexpr int NW = kLocalParts<kMode>;
    constexpr bool kRagged = (kMode == kRev);   // the forward modes cover full segments only
    LocSmem<NW>& S = *reinterpret_cast<LocSmem<NW>*>(smem_raw);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g16 = lane >> 4, l16 = lane & 15;
    const int wi = work_index();
    const int tile = wi % kNTile;
    const int rest = wi / kNTile;
    const int sl = rest % A.NS;                 // local slot of the sequence
    const int s = rest / A.NS;
    const int g = sl / A.R, r = sl % A.R;
    const int v0 = tile * kDVT;
    const int ntiles = A.seg_tokens / kLocTile;
    const int tps = (ntiles + A.R - 1) / A.R;
    const int tile_b = min(ntiles, r * tps), tile_e = min(ntiles, tile_b + tps);
    const int tb = (kMode == kRev ? g + 1 : g) * A.seg_tokens + tile_b * kLocTile;
    int ntok = (tile_e - tile_b) * kLocTile;
    if constexpr (kMode == kRev) ntok = max(0, min(ntok, A.NC * kLocTile - tb));   // the last segment may be shorter

    SeqRsrc P;
    P.k = make_rsrc(seq_rows(A.k, s, A.nh_magic, A.sk), seq_span(A.T, A.rk, kDQK));
    P.v = make_rsrc(seq_rows(A.v, s, A.nh_magic, A.sv), seq_span(A.T, A.rv, kDV));
    if constexpr (kMode != kRev) {
        P.ig = make_rsrc(A.ipre + static_cast<int64_t>(s) * A.T, static_cast<uint32_t>(A.T) * 4);
        P.fg = make_rsrc(A.fpre + static_cast<int64_t>(s) * A.T, static_cast<uint32_t>(A.T) * 4);
    }

    LocRegs rg;
    if (ntok > 0) loc_load<kRagged>(rg, P, tb, v0, tid, A.rk, A.rv);   // first tile, in flight during the gate pass

    float xsum = 0.0f, mloc = 0.0f;   // the slot's last entries
    if constexpr (kMode == kRev) {
        // chunk decays before each chunk of the sub-segment (at most 64 chunks), then the weights
        const int64_t c0 = static_cast<int64_t>(s) * A.NC + tb / kLocTile;
        static_assert(kLocMax / kLocTile <= 64, "one lane per chunk");
        const float dc = (lane < ntok / kLocTile) ? A.decay[c0 + lane] : 1.0f;
        float incl = dc;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const float y = __shfl_up(incl, o, 64);
            if (lane >= o) incl *= y;
        }
        const float before = __shfl_up(incl, 1, 64);
        if (wave == 0) S.w[kLocMax - 64 + lane] = lane ? before : 1.0f;   // moved to registers before the weights land
        xsum = lane63(incl);
        __syncthreads();
        float pref[kLocMax / kThreads];
#pragma unroll
        for (int i = 0; i < kLocMax / kThreads; ++i) pref[i] = S.w[kLocMax - 64 + (i * kThreads + tid) / kLocTile];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kLocMax / kThreads; ++i) {
            const int t = i * kThreads + tid;
            if (t >= ntok) break;
            S.w[t] = pref[i] * A.gd[c0 * kLocTile + t];
            const float wn = pref[i] * A.gw[c0 * kLocTile + t];
            const uint16_t h0 = f32_to_bf16(wn);
            const float r1 = wn - bf16_to_f32(h0);
            const uint16_t h1 = f32_to_bf16(r1);
            S.wb[0][t] = h0;
            S.wb[1][t] = h1;
            S.wb[NW - 1][t] = f32_to_bf16(r1 - bf16_to_f32(h1));
        }
    } else {
        // gates: block-wide prefix sums of logsig(f~) in rounds of 512 tokens (restart tokens add
        // nothing), x_t into LDS, the last restart R, then X over the tokens from R on
        float carry = 0.0f, rmax = -1.0f, xall = -INFINITY;
        for (int j0 = 0; j0 < ntok; j0 += kThreads) {
            const int t = j0 + tid;
            const bool valid = t < ntok;
            const float fv = valid ? bloadf(P.fg, 4 * t, 4 * tb) : 0.0f;
            const float iv = valid ? bloadf(P.ig, 4 * t, 4 * tb) : 0.0f;
            const float lg = valid ? flogsig(fv) : 0.0f;
            const bool rs = (lg == -INFINITY);
            if (rs) rmax = static_cast<float>(t);
            const float incl = wave_incl_sum(rs ? 0.0f : lg);
            if (lane == 63) S.red[0][wave] = incl;
            __syncthreads();
            float before = carry, total = 0.0f;
#pragma unroll
            for (int w2 = 0; w2 < kWaves; ++w2) {
                const float tw = S.red[0][w2];
                if (w2 < wave) before += tw;
                total += tw;
            }
            carry += total;
            const float x = valid ? iv - (before + incl) : -INFINITY;
            if (valid) S.w[t] = x;
            xall = fmaxf(xall, x);
            __syncthreads();   // red[0] is rewritten by the next round
        }
        const float wr = lane63(wave_incl_max(rmax));
        if (lane == 0) S.red[2][wave] = wr;
        __syncthreads();   // the x_t and the restarts of every wave are visible
        float Rf = -1.0f;
#pragma unroll
        for (int w2 = 0; w2 < kWaves; ++w2) Rf = fmaxf(Rf, S.red[2][w2]);
        const int Rl = static_cast<int>(Rf);   // last restart of the sub-segment, -1: none
        float xmax = xall;   // no restart: the maximum over every token
        if (Rl >= 0) {       // block-uniform: only the tokens from the restart on
            xmax = -INFINITY;
            for (int t = Rl + tid; t < ntok; t += kThreads) xmax = fmaxf(xmax, S.w[t]);
        }
        const float wm = lane63(wave_incl_max(xmax));
        if (lane == 0) S.red[1][wave] = wm;
        __syncthreads();
        float X = -INFINITY;
#pragma unroll
        for (int w2 = 0; w2 < kWaves; ++w2) X = fmaxf(X, S.red[1][w2]);
        for (int t = tid; t < ntok; t += kThreads) {
            const float wv = (t < Rl || X == -INFINITY) ? 0.0f : fexp(S.w[t] - X);
            S.w[t] = wv;
            const uint16_t hi = f32_to_bf16(wv);
            const float rest = wv - bf16_to_f32(hi);
            const uint16_t lo = f32_to_bf16(rest);
            S.wb[0][t] = hi;
            S.wb[1][t] = lo;
            if constexpr (NW == 3) S.wb[2][t] = f32_to_bf16(rest - bf16_to_f32(lo));
        }
        mloc = carry + X;   // -inf for an empty sub-segment
        xsum = Rl >= 0 ? -INFINITY : carry;   // sum of logsig(f~)
    }

    // contraction: wave (dh, vg) owns C[128 dh + 0..127][32 vg + 0..31] as 8 x 2 tiles; it also
    // accumulates n over its d tiles 2 vg and 2 vg + 1
    const int dh = wave >> 2, vg = wave & 3;
    f32x4_t Cacc[8][2];
    f32x4_t nacc[2];
#pragma unroll
    for (int q = 0; q < 8; ++q) Cacc[q][0] = Cacc[q][1] = f32x4_t{};
    nacc[0] = nacc[1] = f32x4_t{};
    const int nt = ntok / kLocTile;
    if (nt > 0) {
        loc_store(S.Kt[0], S.Vt[0], rg, tid);
        if (nt > 1) loc_load<kRagged>(rg, P, tb + kLocTile, v0, tid, A.rk, A.rv);
    }
    for (int i = 0; i < nt; ++i) {
        __syncthreads();   // tile i and the weights are visible; the other buffer's readers are done
        if (i + 1 < nt) {
            loc_store(S.Kt[(i + 1) & 1], S.Vt[(i + 1) & 1], rg, tid);
            if (i + 2 < nt) loc_load<kRagged>(rg, P, tb + (i + 2) * kLocTile, v0, tid, A.rk, A.rv);
        }
        const uint16_t* Kt = S.Kt[i & 1];
        const uint16_t* Vt = S.Vt[i & 1];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            const int t0 = i * kLocTile + 32 * ks + 8 * g16;   // this lane's 8 k slots
            const f32x4_t wa0 = *reinterpret_cast<const f32x4_t*>(&S.w[t0]);
            const f32x4_t wa1 = *reinterpret_cast<const f32x4_t*>(&S.w[t0 + 4]);
            const float wv[8] = {wa0[0], wa0[1], wa0[2], wa0[3], wa1[0], wa1[1], wa1[2], wa1[3]};
            u32x4_t Vw[2], Vl[2];
#pragma unroll
            for (int vt = 0; vt < 2; ++vt) {
                const u32x4_t raw = *reinterpret_cast<const u32x4_t*>(&Vt[(32 * vg + 16 * vt + l16) * kLocP + 32 * ks + 8 * g16]);
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const float x0 = lo_f32(raw[u]) * wv[2 * u], x1 = hi_f32(raw[u]) * wv[2 * u + 1];
                    Vw[vt][u] = pack_bf16x2(x0, x1);
                    if constexpr (kHiLo) Vl[vt][u] = pack_bf16x2(x0 - lo_f32(Vw[vt][u]), x1 - hi_f32(Vw[vt][u]));
                }
            }
            const uint16_t* kb = &Kt[(128 * dh + l16) * kLocP + 32 * ks + 8 * g16];
            u32x4_t a[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) a[q] = *reinterpret_cast<const u32x4_t*>(kb + 16 * q * kLocP);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                Cacc[q][0] = mfma16(a[q], Vw[0], Cacc[q][0]);
                Cacc[q][1] = mfma16(a[q], Vw[1], Cacc[q][1]);
                if constexpr (kHiLo) {
                    Cacc[q][0] = mfma16(a[q], Vl[0], Cacc[q][0]);
                    Cacc[q][1] = mfma16(a[q], Vl[1], Cacc[q][1]);
                }
            }
            // n over d tiles 2 vg and 2 vg + 1 (rows re-read by address: no wave-dependent branch)
            const u32x4_t wa = (l16 < NW) ? *reinterpret_cast<const u32x4_t*>(&S.wb[NW == 2 ? l16 & 1 : l16 % NW][t0])
                                          : u32x4_t{0u, 0u, 0u, 0u};
#pragma unroll
            for (int e = 0; e < 2; ++e)
                nacc[e] = mfma16(wa, *reinterpret_cast<const u32x4_t*>(kb + 16 * (2 * vg + e) * kLocP), nacc[e]);
        }
    }

    // slot (s, local slot sl): C [DQK x DV] row-major, then n, m_loc, logsig sum
    MLSTM_CHECK(s < A.S && sl < A.NS && ntok <= kLocMax, kDbgChunkMfma);
    float* slot = A.ws + (static_cast<int64_t>(s) * A.NS + sl) * kSlotFloats;
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
        for (int vt = 0; vt < 2; ++vt)
            *reinterpret_cast<f32x4_t*>(slot + slot_c4(32 * dh + 4 * q + g16, v0 + 32 * vg + 16 * vt + l16)) = Cacc[q][vt];
    if (tile == 0) {
        if (g16 == 0) {
#pragma unroll
            for (int e = 0; e < 2; ++e)
                slot[kDQK * kDV + 128 * dh + 16 * (2 * vg + e) + l16] =
                    nacc[e][0] + (NW == 3 ? nacc[e][1] + nacc[e][2] : nacc[e][1]);
        }
        if (tid == 0) {
            slot[kDQK * kDV + kDQK] = mloc;
            slot[kDQK * kDV + kDQK + 1] = xsum;
        }
    }
}

// Running entry states from the local (sub-)segment states, in place: the last slot of segment g
// (slot g R + R - 1) receives the state after local slots 0..g R + R - 1, the entry state of
// segment g + 1; the other sub-segment slots are only read.
__global__ void __launch_bounds__(256) combine_kernel(float* ws, const float* C0, const float* n0, const float* m0,
                                                      int NS, int R) {
    const int s = blockIdx.y;
    float* base = ws + static_cast<int64_t>(s) * NS * kSlotFloats;
    // scalar chain of entry max states (every block computes it; block 0 stores it)
    float m_in = m0 ? m0[s] : 0.0f;
    constexpr int kE4 = (kDQK * kDV + kDQK) / 4;
    const int e4 = blockIdx.x * blockDim.x + threadIdx.x;
    float4 cur = make_float4(0.f, 0.f, 0.f, 0.f);
    if (e4 < kE4) {
        if (e4 < kDQK * kDV / 4) {
            if (C0) {
                // slot float4 e4 holds rows 4 (e4 / DV) + 0..3 of column e4 % DV; C0 is row-major
                const float* c0 = C0 + static_cast<int64_t>(s) * kDQK * kDV + static_cast<int64_t>(4 * (e4 / kDV)) * kDV + e4 % kDV;
                cur = make_float4(c0[0], c0[kDV], c0[2 * kDV], c0[3 * kDV]);
            }
        } else if (n0) {
            cur = reinterpret_cast<const float4*>(n0 + static_cast<int64_t>(s) * kDQK)[e4 - kDQK * kDV / 4];
        }
    }
    // slots in batches: all loads of a batch are issued before its dependent chain of updates
    constexpr int kBatch = 8;
    for (int g0 = 0; g0 < NS; g0 += kBatch) {
        const int nbat = min(kBatch, NS - g0);
        float4 loc[kBatch];
        float mloc[kBatch], gs[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (u < nbat) {
                const float* slot = base + static_cast<int64_t>(g0 + u) * kSlotFloats;
                mloc[u] = slot[kDQK * kDV + kDQK];
                gs[u] = slot[kDQK * kDV + kDQK + 1];
                if (e4 < kE4) loc[u] = reinterpret_cast<const float4*>(slot)[e4];
            }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (u < nbat) {
                float* slot = base + static_cast<int64_t>(g0 + u) * kSlotFloats;
                // a restart inside the slot (gs = -inf) drops the running state; an empty slot
                // (m_loc = -inf) adds nothing
                const float carried = gs[u] + m_in;
                const float m_new = fmaxf(carried, mloc[u]);
                const float a = (carried == -INFINITY) ? 0.0f : expf(carried - m_new);
                const float b = (mloc[u] == -INFINITY) ? 0.0f : expf(mloc[u] - m_new);
                const bool entry = ((g0 + u) % R) == R - 1;
                if (e4 < kE4) {
                    cur.x = a * cur.x + b * loc[u].x;
                    cur.y = a * cur.y + b * loc[u].y;
                    cur.z = a * cur.z + b * loc[u].z;
                    cur.w = a * cur.w + b * loc[u].w;
                    if (entry) reinterpret_cast<float4*>(slot)[e4] = cur;
                }
                if (entry && blockIdx.x == 0 && threadIdx.x == 0) slot[kDQK * kDV + kDQK + 2] = m_new;
                m_in = m_new;
            }
        }
    }
}

// q, k, v strides of a call: the caller's (elements; batch, head, token for each), or contiguous
// [B, NH, T, D] rows; the kernels take {batch - NH head, head} per matrix (see seq_rows)
void set_strides(const ChunkArgs& a, uint32_t& nh_magic, int64_t* sq, int64_t* sk, int64_t* sv, uint32_t* rq,
                 uint32_t* rk, uint32_t* rv) {
    nh_magic = a.NH > 1 ? static_cast<uint32_t>((uint64_t(1) << 32) / static_cast<uint64_t>(a.NH) + 1) : 0u;
    const int64_t T = a.T, NH = a.NH;
    const int64_t st[9] = {NH * T * kDQK, T * kDQK, kDQK, NH * T * kDQK, T * kDQK, kDQK, NH * T * kDV, T * kDV, kDV};
    const int64_t* x = a.strides ? a.strides : st;
    if (sq) {
        sq[0] = x[0] - NH * x[1];
        sq[1] = x[1];
    }
    sk[0] = x[3] - NH * x[4];
    sk[1] = x[4];
    sv[0] = x[6] - NH * x[7];
    sv[1] = x[7];
    if (rq) *rq = static_cast<uint32_t>(x[2] * 2);
    *rk = static_cast<uint32_t>(x[5] * 2);
    *rv = static_cast<uint32_t>(x[8] * 2);
}

hipError_t launch_chunks(const ChunkKernelArgs& a, int S, hipStream_t stream) {
    const size_t lds = sizeof(Smem);
    auto kern = chunk_mfma_kernel;
    static std::atomic<uint64_t> raised{0};
    hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(kern), lds, raised);
    if (e != hipSuccess) return e;
    const dim3 grid(static_cast<unsigned>(S * a.G * kNTile));
    hipLaunchKernelGGL(kern, grid, dim3(kThreads), lds, stream, a);
    return hipGetLastError();
}

template <LocalMode kMode>
hipError_t launch_local(const LocalArgs& a, int S, hipStream_t stream) {
    const size_t lds = sizeof(LocSmem<kLocalParts<kMode>>);
    static std::atomic<uint64_t> raised{0};
    auto kern = local_state_kernel<kMode>;
    hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(kern), lds, raised);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(S * a.NS * kNTile)), dim3(kThreads), lds, stream, a);
    return hipGetLastError();
}

// sub-segments of a local segment: at most kLocMax tokens each
int local_subsegments(int seg_tokens) { return (seg_tokens + kLocMax - 1) / kLocMax; }

}  // namespace

bool chunk_mfma_supported(mlstm_dtype dt, int DQK, int DV, int L) {
    return dt == MLSTM_BF16 && DQK == kDQK && DV == kDV && (L == 64 || L == 128);
}

int chunk_mfma_segments(int B, int NH, int T, int L) {
    const int S = B * NH;
    const int nc = (T + L - 1) / L;
    if (nc <= 1) return 1;
    const int wgs = S * kNTile;
    constexpr int kTargetWGs = 256;
    int G = (kTargetWGs + wgs - 1) / wgs;
    if (G > nc / 2) G = nc / 2;   // at least two chunks per segment
    if (G < 1) G = 1;
    const int seg = (nc + G - 1) / G;
    return (nc + seg - 1) / seg;
}

size_t chunk_mfma_workspace_bytes(int B, int NH, int T, int DQK, int DV, int L) {
    (void)DQK;
    (void)DV;
    const int G = chunk_mfma_segments(B, NH, T, L);
    if (G <= 1) return 0;
    const int nc = (T + L - 1) / L;
    const int seg_tokens = ((nc + G - 1) / G) * L;
    return static_cast<size_t>(B) * NH * (G - 1) * local_subsegments(seg_tokens) * kSlotFloats * sizeof(float);
}

// ---- the segment schedule ---------------------------------------------------------------------
SegmentShape segment_shape(int B, int NH, int T, int L, bool use_segments) {
    SegmentShape sh{};
    const int nc = (T + L - 1) / L;
    sh.G = (use_segments && nc > 0) ? chunk_mfma_segments(B, NH, T, L) : 1;
    sh.seg_chunks = sh.G > 1 ? (nc + sh.G - 1) / sh.G : nc;
    sh.R = sh.G > 1 ? local_subsegments(sh.seg_chunks * L) : 1;
    return sh;
}

hipError_t launch_segment_states(const ChunkArgs& a, int L, const SegmentShape& sh, float* seg, bool hilo,
                                 hipStream_t stream) {
    if (sh.G <= 1) return hipSuccess;
    const int S = a.B * a.NH;
    LocalArgs la{};
    la.k = static_cast<const uint16_t*>(a.k);
    la.v = static_cast<const uint16_t*>(a.v);
    set_strides(a, la.nh_magic, nullptr, la.sk, la.sv, nullptr, &la.rk, &la.rv);
    la.ipre = a.ipre;
    la.fpre = a.fpre;
    la.ws = seg;
    la.S = S;
    la.T = a.T;
    la.NS = (sh.G - 1) * sh.R;
    la.R = sh.R;
    la.seg_tokens = sh.seg_chunks * L;
    hipError_t e = hilo ? launch_local<kFwdHiLo>(la, S, stream) : launch_local<kFwd>(la, S, stream);
    if (e != hipSuccess) return e;
    constexpr int kE4 = (kDQK * kDV + kDQK) / 4;
    hipLaunchKernelGGL(combine_kernel, dim3((kE4 + 255) / 256, S), dim3(256), 0, stream, seg, a.C0, a.n0, a.m0, la.NS,
                       sh.R);
    return hipGetLastError();
}

hipError_t launch_reverse_local(const ReverseLocal& a, hipStream_t stream) {
    LocalArgs la{};
    la.k = a.q;
    la.v = a.dh;
    la.sk[1] = static_cast<int64_t>(a.T) * kDQK;   // contiguous rows (nh_magic 0: the sequence index alone)
    la.sv[1] = static_cast<int64_t>(a.T) * kDV;
    la.rk = kDQK * 2;
    la.rv = kDV * 2;
    la.ws = a.seg;
    la.S = a.S;
    la.T = a.T;
    la.NS = a.NS;
    la.R = a.R;
    la.seg_tokens = a.seg_chunks * kLocTile;
    la.gd = a.gd;
    la.gw = a.gw;
    la.decay = a.decay;
    la.NC = a.NC;
    return launch_local<kRev>(la, a.S, stream);
}

hipError_t launch_chunk_mfma(const ChunkArgs& a, void* workspace, size_t workspace_bytes, hipStream_t stream) {
    const int S = a.B * a.NH;
    const bool use_segments =
        workspace != nullptr && workspace_bytes >= chunk_mfma_workspace_bytes(a.B, a.NH, a.T, a.DQK, a.DV, a.L);
    const SegmentShape sh = segment_shape(a.B, a.NH, a.T, a.L, use_segments);

    ChunkKernelArgs k{};
    k.q = static_cast<const uint16_t*>(a.q);
    k.k = static_cast<const uint16_t*>(a.k);
    k.v = static_cast<const uint16_t*>(a.v);
    set_strides(a, k.nh_magic, k.sq, k.sk, k.sv, &k.rq, &k.rk, &k.rv);
    k.ipre = a.ipre;
    k.fpre = a.fpre;
    k.C0 = a.C0;
    k.n0 = a.n0;
    k.m0 = a.m0;
    k.ws = static_cast<float*>(workspace);
    k.S = S;
    k.T = a.T;
    k.G = sh.G;
    k.R = sh.R;
    k.NS = (sh.G - 1) * sh.R;
    // Chunks of 64 tokens for L = 128 too: the result depends on the chunk length only through rounding, and
    // L = 128 did twice the work inside a chunk on the same waves (its own kernel took 2020 us for 4 x 32768
    // tokens from a state against 1857 here, 452 against 405 for 16 x 2048, 18.7 against 17.4 for 100).  The
    // segments, and so the workspace, stay those of the caller's L.
    k.seg_chunks = sh.seg_chunks * (a.L / 64);
    // A chunk that rescales C eagerly has weights exp(x - M_L), and the token with the largest is not rounded at
    // all; with a lazy scale every term of C takes a rounding.  Chunks of 128 tokens rescaled about twice as often
    // as their halves do, so for L = 128 the last chunk, which makes up most of the final state, always does.
    k.eager_chunk = a.L == 128 ? (a.T + 63) / 64 - 1 : -1;
    k.h = static_cast<uint16_t*>(a.h);
    k.CT = a.CT;
    k.nT = a.nT;
    k.mT = a.mT;

    hipError_t e = launch_segment_states(a, a.L, sh, k.ws, false, stream);
    if (e != hipSuccess) return e;
    return launch_chunks(k, S, stream);
}

// ---- fixed scratch for callers that cannot allocate ---------------------------------------------
// The segment slots of mlstm_chunkwise_fwd_noalloc.  Every slot a call reads is written earlier in
// the same call (local pass, then combine), so nothing needs clearing between calls; calls that
// overlap on one device share this array and race.
namespace {
__device__ __attribute__((aligned(256))) unsigned char scratch[kChunkScratchBytes];
constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxScratchDevices] = {};
}  // namespace

hipError_t chunk_scratch(void** ptr) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxScratchDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        // the device address of this device's copy (the host-side name is not a device address)
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

#ifdef MLSTM_DEBUG
MLSTM_DEBUG_READER(debug_flags_chunk_mfma)
#endif

}  // namespace mlstm

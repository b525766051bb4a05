// Chunkwise backward of the mLSTM cell on bf16 MFMA for the xLSTM 7B head shape
// (DQK = 256, DV = 512), chunk length 64: the gradients of sum(h~ . dh) with respect to
// q, k, v, the gate pre-activations and the initial state (C0, n0, m0).
//
// Math.  Per chunk c with entry state (C, n, m_prev) (stabilised by m_prev), the gates of the
// forward (in-chunk prefix sums b, x = i~ - b, last restart R_tau, M_tau, key weights
// w_tau = exp(x_tau - M_L), decay = exp(m_prev - M_L)), g_tau = exp(m_prev - M_tau) and
// floor_tau = exp(-(b_tau + M_tau)) (App. D.1), with q^ = q / sqrt(DQK):
//
//   S = Q^ K^T,  E_ts = exp(x_s - M_t) for R_t <= s <= t (else 0),  St = S o E
//   D_t = g_t (q^_t . n) + sum_s St_ts,  den_t = max(|D_t|, floor_t),  h~_t = N_t / den_t with
//   N_t = g_t (C^T q^_t) + sum_s St_ts v_s
//   U = dH / den (rows),  w_t = -(dh_t . N_t) sign(D_t) / den_t^2  where |D_t| > floor_t, else 0
//   P = E o (U V^T + w 1^T)
//   dq^ = P K + diag(g) (U C^T + w n^T),   dk = P^T Q^ + diag(wkey) (V Gam^T + 1 gam^T),
//   dv  = St^T U + diag(wkey) K Gam,
// where (Gam_c, gam_c) is the gradient reaching chunk c's exit state (C_c, n_c), in the units of
// its stabiliser, from all later chunks; it runs backwards through the state recurrence of
// Eqs. 3-4 in chunk form:
//   Gam_{c-1} = decay_c Gam_c + L_c,   L_c = Q^T diag(g / den) dH,
//   gam_{c-1} = decay_c gam_c + z_c,   z_c = Q^T (g o w) / sqrt(DQK)
// (Gam of the last chunk is zero; Gam_{-1}, gam_{-1} are the gradients of C0 and n0, and
// dm0 = <Gam_{-1}, C0> + gam_{-1} . n0 since the unstabilised state is e^{m0} (C0, n0)).
// The gate gradients follow from the two row sums r_t = q_t . dq_t and c_t = k_t . dk_t:
//   di~_t = c_t,  dlogsig(f~_t) = sum_{t' >= t} (r_t' - c_t'),  df~_t = that times sigmoid(-f~_t)
// (a forget gate of zero, f~ = -inf, is a restart; its own gradient is zero).
//
// dh_t . N_t is formed in fp32 from its two parts, g_t q^_t . (C dh_t) and sum_s St_ts (dh_t . v_s),
// rather than from the forward's rounded h~: where the two terms of dq nearly cancel, the bf16
// rounding of h~ would dominate the result.  The forward's output is not an input.
//
// Passes (one stream, in order):
//   states  the prefill's segment schedule (local pass in the bf16 hi + lo form, combine) for the
//           entry states of segments of several chunks (long enough batches need none)
//   x       a walk over each segment's chunks per 64-row tile of d, holding its 64 x 512 slice of the
//           state in registers: per chunk X = dH C^T on the entry state (complete: the tile holds all
//           of v), the tile's share of q^_t . X_t, then the state update; n and m entering each chunk
//   intra   one workgroup per chunk: gates, S, D, den, dH V^T, w, P, dq (complete), q_t . dq_t; writes
//           St / den and P (transposed, bf16; P as hi + lo) and the per-token scalars the walks need
//   rstates the gradients reaching the exits of the segments: a local pass over each segment but the
//           first (its own contribution, one weighted contraction) and a reverse combine
//   dk      a reverse walk over each segment's chunks per 64-row tile of d, holding its slice of Gam in
//           registers: dk (inter and intra terms, complete), k . dk, then Gam <- decay Gam + L_c, gam;
//           at the first chunk dC0, dn0 and partial sums of dm0
//   dv      the same per 128-column tile of v: dv (inter and intra terms, complete)
//   gates   one workgroup per sequence: the reverse prefix sums of r - c, di~ and df~, dm0
// Neither the states nor Gam nor L_c go to memory (8 + 8 + 4 KB per token and head when they did: the
// three passes that wrote and read them took 5.3 of the 8.3 ms of a 16 x 4096-token training step); the
// two reverse walks each carry Gam because the dk product sums over v and the dv product over d, so one
// slice layout would leave one of them summed across workgroups.
//
// MFMA mapping (16x16x32 bf16, fp32 accumulate): lane (l16, g16) holds A[m = l16][k = 8 g16 + 0..7]
// and B[k = 8 g16 + 0..7][n = l16] and receives D[m = 4 g16 + 0..3][n = l16].  An operand whose
// contraction index is contiguous in memory is one 16-byte row read; otherwise it comes from a
// row-major [k][n] tile in LDS through the transpose read.  Every product is arranged so that its
// output lane holds four consecutive elements of one output row (one 16-byte store).
//
// Rows past the end of the sequence (a partial last chunk) are read through buffer resources with
// the row offset in the range-checked offset, so they read as zero.
#include "chunk_common.h"
#include "launch.h"

namespace mlstm {
namespace {

constexpr int kBL = 64;                                   // tokens per chunk
constexpr int kQP = kDQK + 8;                             // LDS pitch of K rows in the intra pass (528 bytes)
constexpr int kPP = kBL + 8;                              // LDS pitch of [tau][sigma] tiles (144 bytes)
constexpr int64_t kCV = static_cast<int64_t>(kDQK) * kDV; // elements of one state matrix
constexpr int kPart = 8;                                  // partial sums per token of q^ . X and of k . dk
constexpr int kDTile = 64;                                // d rows per workgroup of the x and dk walks
constexpr int kNDT = kDQK / kDTile;                       // their tiles per sequence

struct BwdParams {
    const uint16_t* q;
    const uint16_t* k;
    const uint16_t* v;
    const uint16_t* dh;
    const float* ipre;
    const float* fpre;
    const float* C0;     // NULL: zero initial state (with n0, m0)
    const float* n0;
    const float* m0;
    void* dq;            // [S, T, D] rows, fp32 or bf16 (the passes' kBf16)
    void* dk;
    void* dv;
    float* dip;
    float* dfp;
    float* dC0;          // NULL: not requested (with dn0, dm0)
    float* dn0;
    float* dm0;
    float* seg;          // segment slots: of the forward states, then of the gradients (NULL when G == 1)
    float* X;            // S x T x DQK: X = dH C^T on the entry states
    float* nst;          // S x NC x DQK: n entering each chunk
    float* mst;          // S x NC: m entering each chunk
    float* decay;        // S x NC: decay of each chunk
    // per token, padded to whole chunks (S x NC x 64, zero past T): key weight, g / den / sqrt(DQK),
    // g w / sqrt(DQK)
    float* wk;
    float* gd;
    float* gw;
    uint16_t* SnT;       // S x NC x 64 x 64: (St / den)^T [sigma][tau]
    uint16_t* PT;        // S x NC x 2 x 64 x 64: P^T [sigma][tau] as bf16 hi, lo
    float* qx;           // S x T x kPart: partial sums of q^ . X
    float* kdk;          // S x T x kPart: partial sums of k . dk
    float* r;            // S x T: q . dq
    float* dmp;          // S x kNDT: partial sums of dm0
    int S;
    int T;
    int NC;
    int G;               // segments per sequence
    int R;               // local sub-segments per segment
    int NS;              // segment slots per sequence, (G - 1) R
    int seg_chunks;      // chunks per segment (the last may be shorter)
};

__device__ __forceinline__ u32x4_t lds16(const uint16_t* p) { return *reinterpret_cast<const u32x4_t*>(p); }
// operand whose contraction index runs along rows: lane gets row r0 + l16, k = k0 + 8 g16 + 0..7
__device__ __forceinline__ u32x4_t row_op(const uint16_t* base, int pitch, int r0, int k0, int lane) {
    return lds16(base + (r0 + (lane & 15)) * pitch + k0 + 8 * (lane >> 4));
}
// operand from a row-major [k][n] LDS tile: lane gets column n0 + l16, k = k0 + 8 g16 + 0..7
__device__ __forceinline__ u32x4_t tr_op(const uint16_t* base, int pitch, int k0, int n0, int lane) {
    const int g16 = lane >> 4, l16 = lane & 15;
    const uint16_t* p = base + (k0 + 8 * g16 + (l16 >> 2)) * pitch + n0 + 4 * (l16 & 3);
    return cat(tr_read(p), tr_read(p + 4 * pitch));
}
__device__ __forceinline__ float bf_at(const u32x4_t& w, int e) {
    return (e & 1) ? hi_f32(w[e >> 1]) : lo_f32(w[e >> 1]);
}
// eight bf16 values times w, rounded once
__device__ __forceinline__ u32x4_t scale8(const u32x4_t& x, float w) {
    u32x4_t o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = pack_bf16x2(lo_f32(x[i]) * w, hi_f32(x[i]) * w);
    return o;
}
__device__ __forceinline__ float wave_total(float x) { return lane63(wave_incl_sum(x)); }
__device__ __forceinline__ float dot4(const u32x2_t& a, const f32x4_t& b) {
    return lo_f32(a[0]) * b[0] + hi_f32(a[0]) * b[1] + lo_f32(a[1]) * b[2] + hi_f32(a[1]) * b[3];
}
// eight consecutive fp32 values (two accumulator tiles of a pair) as a bf16 operand, and what it drops
__device__ __forceinline__ u32x4_t pack8(const f32x4_t& a, const f32x4_t& b) {
    return u32x4_t{pack_bf16x2(a[0], a[1]), pack_bf16x2(a[2], a[3]), pack_bf16x2(b[0], b[1]), pack_bf16x2(b[2], b[3])};
}
__device__ __forceinline__ u32x4_t pack8_lo(const f32x4_t& a, const f32x4_t& b, const u32x4_t& h) {
    return u32x4_t{pack_bf16x2(a[0] - lo_f32(h[0]), a[1] - hi_f32(h[0])), pack_bf16x2(a[2] - lo_f32(h[1]), a[3] - hi_f32(h[1])),
                   pack_bf16x2(b[0] - lo_f32(h[2]), b[1] - hi_f32(h[2])), pack_bf16x2(b[2] - lo_f32(h[3]), b[3] - hi_f32(h[3]))};
}

// ---- gates of one chunk (one wave, lane = row) -------------------------------------------------
struct BGate {
    float x, M, g, fl, wk;
    int R;
};
__device__ __forceinline__ void bwd_gates(__amdgpu_buffer_rsrc_t ig, __amdgpu_buffer_rsrc_t fg, int T, int t0,
                                          float m_prev, int lane, BGate& G, float& decay) {
    const int t = t0 + lane;
    const bool ok = t < T;
    const uint32_t off = static_cast<uint32_t>(t) * 4u;
    const float fv = bloadf(fg, off, 0), iv = bloadf(ig, off, 0);
    const float lg = ok ? flogsig(fv) : 0.0f;
    const bool rs = (lg == -INFINITY);
    const bool any = __builtin_amdgcn_ballot_w64(rs) != 0;
    const float b = wave_incl_sum(rs ? 0.0f : lg);
    const float x = ok ? iv - b : -INFINITY;
    float r = -1.0f, p;
    if (any) {
        r = wave_incl_max(rs ? static_cast<float>(lane) : -1.0f);
        p = wave_seg_incl_max(x, rs);
    } else {
        p = wave_incl_max(x);
    }
    const float pL = lane63(p), rL = lane63(r);
    const bool restart = rL >= 0.0f;
    const float ML = restart ? pL : fmaxf(m_prev, pL);
    const bool fresh = r >= 0.0f;
    const float M = fresh ? p : fmaxf(m_prev, p);
    G.x = x;
    G.M = M;
    G.R = static_cast<int>(r);
    G.g = (fresh || M == -INFINITY) ? 0.0f : fexp(m_prev - M);
    G.fl = fexp(-(b + M));
    const bool none = (x == -INFINITY) || (static_cast<float>(lane) < rL);
    G.wk = none ? 0.0f : fexp(x - ML);
    decay = (restart || ML == -INFINITY || m_prev == -INFINITY) ? 0.0f : fexp(m_prev - ML);
}

// Per-lane accesses of the walks go through range-checked buffers instead of branches (rows past the end
// read as zero, and their stores are dropped), and the next chunk's loads are issued in every chunk (the
// last one repeats a chunk): with no branch between them the compiler counts the loads in flight and waits
// for the ones it needs, where behind a branch it waits for all (1074 -> 786 us for the dv walk of
// 16 x 4096 tokens).
constexpr uint32_t kNoStore = 0xFFFFFFF0u;   // an offset outside every buffer
__device__ __forceinline__ u32x2_t bload64(__amdgpu_buffer_rsrc_t r, uint32_t voff) {
    return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(r, voff, 0, 0));
}
__device__ __forceinline__ void bstore128(__amdgpu_buffer_rsrc_t r, uint32_t voff, const f32x4_t& x) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, x), r, voff, 0, 0);
}
// four consecutive gradients of a row at element offset e of a [T, D] matrix, fp32 or rounded once to bf16
template <bool kBf16>
__device__ __forceinline__ void store_grad(__amdgpu_buffer_rsrc_t r, uint32_t e, const f32x4_t& x) {
    if constexpr (kBf16)
        __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3])}, r, e * 2u, 0, 0);
    else
        bstore128(r, e * 4u, x);
}
template <bool kBf16>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t grad_rsrc(void* p, int64_t row0, int T, int D) {
    constexpr int eb = kBf16 ? 2 : 4;
    return make_rsrc(static_cast<unsigned char*>(p) + row0 * D * eb, static_cast<uint32_t>(T) * static_cast<uint32_t>(D * eb));
}
__device__ __forceinline__ void bstoref(__amdgpu_buffer_rsrc_t r, uint32_t voff, float x) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), r, voff, 0, 0);
}

// ---- staging of the walks -----------------------------------------------------------------------
// A walk's chunk operands in LDS: [64][512] rows at a 1056-byte pitch (16 consecutive rows fall in
// different banks), and transposed matrices (rows = columns of the source, 64 tau at a 144-byte pitch),
// transposed on the matrix cores by a one-hot product (exact) from pieces in the A-operand layout.
// The rows of a transposed matrix are stored in pair order, pair_row: the 16 rows 8 i + 4 e + j
// (i, j = 0..3) that the A operand of accumulator tile e of a pair reads are consecutive.
constexpr int kRP = kDV + 16;    // pitch of [64][512] rows
constexpr int kTP = kBL + 8;     // pitch of the transposed matrices, and of [64][64] tiles
__device__ __forceinline__ int pair_row(int v) {
    return (v & ~31) | (((v >> 2) & 1) << 4) | (((v >> 3) & 3) << 2) | (v & 3);
}

// rows t0 .. t0 + 63 of a [T][512] bf16 matrix, eight 16-byte pieces per thread
__device__ __forceinline__ u32x4_t load_row512(__amdgpu_buffer_rsrc_t m, int t0, int i, int tid) {
    return bload128(m, static_cast<uint32_t>(t0 + (tid >> 6) + 8 * i) * (kDV * 2) + 16 * (tid & 63), 0);
}
__device__ __forceinline__ void load_rows512(u32x4_t (&r)[8], __amdgpu_buffer_rsrc_t m, int t0, int tid) {
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = load_row512(m, t0, i, tid);
}
__device__ __forceinline__ void store_rows512(uint16_t* dst, const u32x4_t (&r)[8], int tid) {
#pragma unroll
    for (int i = 0; i < 8; ++i) *reinterpret_cast<u32x4_t*>(dst + ((tid >> 6) + 8 * i) * kRP + 8 * (tid & 63)) = r[i];
}
// pieces of 16 tau x 32 columns: wave w takes the tau block w % 4 and the N column blocks N (w / 4) + i, so
// that the two 64-byte halves of a memory line are requested by one wave, one after the other
template <int N>
__device__ __forceinline__ u32x4_t load_piece(__amdgpu_buffer_rsrc_t m, int row_bytes, int t0, int i, int wave, int lane) {
    return bload128(m, static_cast<uint32_t>(t0 + 16 * (wave & 3) + (lane & 15)) * row_bytes +
                           (32 * (N * (wave >> 2) + i) + 8 * (lane >> 4)) * 2, 0);
}
template <int N>
__device__ __forceinline__ void load_pieces(u32x4_t (&r)[N], __amdgpu_buffer_rsrc_t m, int row_bytes, int t0, int wave,
                                            int lane) {
#pragma unroll
    for (int i = 0; i < N; ++i) r[i] = load_piece<N>(m, row_bytes, t0, i, wave, lane);
}
template <int N>
__device__ __forceinline__ void store_transposed(uint16_t* dst, const u32x4_t (&r)[N], int wave, int lane) {
    u32x4_t E[2];
    onehot_pair(E, lane);
    const int l16 = lane & 15, g16 = lane >> 4;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const f32x4_t d = mfma16(r[i], E[h], f32x4_t{});
            const int row = pair_row(32 * (N * (wave >> 2) + i) + 16 * h + l16);
            MLSTM_CHECK(row < 64 * N, kDbgChunkBwd);
            *reinterpret_cast<u32x2_t*>(dst + row * kTP + 16 * (wave & 3) + 4 * g16) =
                u32x2_t{pack_bf16x2(d[0], d[1]), pack_bf16x2(d[2], d[3])};
        }
}

// ---- walks over a 64-row tile of d (x, dk) -------------------------------------------------------
// Wave w = 2 vq + dp owns the 32 x 128 block d = 64 tile + 32 dp + 0..31, v = 128 vq + 0..127 of the
// state (C or Gam) as accumulator tiles (dt, pp, e): lane (l16, g16) holds state[d = 32 dp + 16 dt + l16]
// [v = 128 vq + 32 pp + 8 g16 + 4 e + j], j = 0..3, so the two tiles of a pair give a lane eight consecutive
// v: the A operand of (state R^T)[d][tau] = sum_v state[d][v] R[tau][v] with 16-byte reads of the rows R.
// The product's partial sums over vq meet in LDS: the wave (dp, vq) finishes the tau tile vq.  X[dt][i] is
// the tau tile (vq + i) % 4, so that the tile a wave keeps has a fixed register (a choice by wave would
// put the array into scratch memory).
typedef f32x4_t DState[2][4][2];

// issue(pp) is called once per 32 v: the next chunk's loads go out between the products (issued together
// before them, 18 loads per wave kept every wave from its products for about 2300 cycles of a chunk).
template <bool kHiLo, class F>
__device__ __forceinline__ void dtile_product(f32x4_t (&X)[2][4], const DState& C, const uint16_t* rows, int vq, int lane,
                                              F issue) {
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) X[dt][tb] = f32x4_t{};
#pragma unroll
    for (int pp = 0; pp < 4; ++pp) {
        u32x4_t b[4];
#pragma unroll
        for (int tb = 0; tb < 4; ++tb) b[tb] = row_op(rows, kRP, 16 * ((vq + tb) & 3), 128 * vq + 32 * pp, lane);
        issue(pp);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
            const u32x4_t ah = pack8(C[dt][pp][0], C[dt][pp][1]);
#pragma unroll
            for (int tb = 0; tb < 4; ++tb) X[dt][tb] = mfma16(ah, b[tb], X[dt][tb]);
            if constexpr (kHiLo) {
                const u32x4_t al = pack8_lo(C[dt][pp][0], C[dt][pp][1], ah);
#pragma unroll
                for (int tb = 0; tb < 4; ++tb) X[dt][tb] = mfma16(al, b[tb], X[dt][tb]);
            }
        }
    }
}
// exchange of the partial products: wave w's X[dt][i], i = 1..3, at ex[((3 w + i - 1) 2 + dt) 64 + lane]
constexpr int kExBytes = kWaves * 3 * 2 * 64 * 16;
static_assert(kExBytes <= 64 * kRP * 2, "the exchange lives in the rows it was computed from");
__device__ __forceinline__ void dtile_give(f32x4_t* ex, const f32x4_t (&X)[2][4], int wave, int lane) {
#pragma unroll
    for (int i = 1; i < 4; ++i)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) ex[((3 * wave + i - 1) * 2 + dt) * 64 + lane] = X[dt][i];
}
__device__ __forceinline__ void dtile_take(f32x4_t (&Y)[2], const f32x4_t* ex, const f32x4_t (&X)[2][4], int vq, int dp,
                                           int lane) {
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) {
        Y[dt] = X[dt][0];
#pragma unroll
        for (int i = 1; i < 4; ++i) Y[dt] += ex[((3 * (2 * ((vq - i) & 3) + dp) + i - 1) * 2 + dt) * 64 + lane];
    }
}
// state += (M^T)[v][tau] B[tau][d] over 32 tau: A = rows of the transposed matrix in pair order, B in NB
// parts (hi, lo) per d tile
template <int NB, class F>
__device__ __forceinline__ void dtile_update(DState& C, const uint16_t* Mt, const u32x4_t (&b)[NB][2], int vq, int ks,
                                             int lane, F issue) {
#pragma unroll
    for (int pp = 0; pp < 4; ++pp) {
        issue(4 * ks + pp);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const u32x4_t a = row_op(Mt, kTP, 128 * vq + 32 * pp + 16 * e, 32 * ks, lane);
#pragma unroll
            for (int p = 0; p < NB; ++p)
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) C[dt][pp][e] = mfma16(a, b[p][dt], C[dt][pp][e]);
        }
    }
}
// The order of one dtile_update (half a chunk's) with its kTr transpose reads and kProducts products per pp: the
// next chunk's load of a pp before its products, the operands one pp ahead.  Left to itself the compiler puts the
// loads last, and the next chunk waits for them (16 x 4096 tokens: x walk 854 us, 845 in this order; dk walk 820, 791).
template <int kTr, int kProducts>
__device__ __forceinline__ void dtile_update_order() {
    __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, kTr + 4, 0);
    __builtin_amdgcn_sched_group_barrier(0x8, kProducts, 0);
    __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x8, kProducts, 0);
    __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    __builtin_amdgcn_sched_group_barrier(0x8, kProducts, 0);
    __builtin_amdgcn_sched_group_barrier(0x20, 1, 0);
    __builtin_amdgcn_sched_group_barrier(0x8, kProducts, 0);
    __builtin_amdgcn_sched_barrier(0);
}
// the tile from a segment slot (four rows interleaved: element (d, v) at slot_c4(d / 4, v) + d % 4)
__device__ __forceinline__ void dtile_from_slot(DState& C, const float* slot, int d0, int vq, int lane) {
    const int l16 = lane & 15, g16 = lane >> 4;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt) {
        const int d = d0 + 16 * dt + l16;
#pragma unroll
        for (int pp = 0; pp < 4; ++pp)
#pragma unroll
            for (int e = 0; e < 2; ++e)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    C[dt][pp][e][j] = slot[slot_c4(d / 4, 128 * vq + 32 * pp + 8 * g16 + 4 * e + j) + d % 4];
    }
}
__device__ __forceinline__ int64_t dtile_c0(int d0, int dt, int vq, int pp, int e, int lane) {
    return static_cast<int64_t>(d0 + 16 * dt + (lane & 15)) * kDV + 128 * vq + 32 * pp + 8 * (lane >> 4) + 4 * e;
}

// The thread's lane quantities re-derived from an opaque copy of its index, in every chunk: otherwise the
// compiler holds every lane-dependent address across the chunk loop and spills.
#define MLSTM_OPAQUE_LANES(outer)               \
    int tid = (outer);                          \
    asm volatile("" : "+v"(tid));               \
    const int lane = tid & 63;                  \
    const int g16 = lane >> 4, l16 = lane & 15

// ---- x: X = dH C^T on the entry states -----------------------------------------------------------
// One workgroup of 8 waves per (sequence, 64-row d tile, segment), with the gate phase and lazy scale of
// chunk_mfma_kernel (C = C_acc e^{s}).  Per chunk: X^T = C dH^T with C as a bf16 pair hi + lo, then
// C += (w e^{-s} K)^T V with the weighted keys as a bf16 pair (products to about 2^-17 rather than the 2^-9
// of one rounding, because the backward's gradients can cancel against the state).  The
// weights go on K, whose tile is 64 columns wide, rather than on V: half the operand reads of the update.
// n is summed in fp32 from the fp32 weights and the keys themselves: q . n decides the branch |D| > floor, and
// with n from the rounded pair (weights times e^{-s}, whose exponent is up to 20 larger) three times as many rows
// of 1 x 2048-token calls fell on the wrong side of it.
struct XSmem {
    uint16_t Vt[kDV * kTP];        // the chunk's V^T, rows in pair order
    uint16_t dH[kBL * kRP];        // the chunk's dH rows, then the exchange of the partial products
    uint16_t Kw[2][kBL * 68];      // w e^{-s} K rows of this d tile as bf16 hi, lo (136-byte pitch)
    GateBuf<true> G[2];        // by chunk parity
};
static_assert(sizeof(XSmem) <= 160 * 1024, "LDS budget");
// the waves' partial sums of n (kWaves x 64 floats) take the place of the dH rows behind the exchange
static_assert(kExBytes + kWaves * kDTile * 4 <= 64 * kRP * 2, "n partials");

// x[0..7] of a lane are its columns 8 (lane % 8) + 0..7 of row lane / 8; the sum over the eight rows of column
// 8 (lane % 8) + rows8_col(lane), one column per lane (each step halves the columns a lane still sums)
__device__ __forceinline__ int rows8_col(int lane) { return 4 * (lane >> 5) + 2 * ((lane >> 4) & 1) + ((lane >> 3) & 1); }
__device__ __forceinline__ float rows8_sum(const float (&x)[8], int lane) {
    float y[4], z[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {   // lanes 0..31 keep columns 0..3, lanes 32..63 columns 4..7
        const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x[i]), __float_as_uint(x[i + 4]), false, false);
        y[i] = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {   // even rows of 16 lanes keep the first two of their columns, odd ones the others
        const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(y[i]), __float_as_uint(y[i + 2]), false, false);
        z[i] = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    }
    const bool odd = (lane & 8) != 0;
    const float keep = odd ? z[1] : z[0], give = odd ? z[0] : z[1];
    return keep + __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, give), 0x128, 0xf, 0xf, false));   // row_ror:8
}

__global__ void __launch_bounds__(kThreads, 1) bwd_x_kernel(BwdParams A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    XSmem& S = *reinterpret_cast<XSmem*>(smem_raw);
    constexpr int KP = 68;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int dp = wave & 1, vq = wave >> 1;
    const bool gate_wave = (wave == kGateWave);

    const int wi = work_index();
    const int tile = wi % kNDT;
    const int g = (wi / kNDT) % A.G;
    const int s = wi / kNDT / A.G;
    const int d0 = kDTile * tile + 32 * dp;   // first d of this wave
    const int c_begin = g * A.seg_chunks;
    const int c_end = min(A.NC, c_begin + A.seg_chunks);
    MLSTM_CHECK(s < A.S, kDbgChunkBwd);
    const int64_t st = static_cast<int64_t>(s) * A.T;

    SeqRsrc P;
    P.k = make_rsrc(A.k + st * kDQK, static_cast<uint32_t>(A.T) * (kDQK * 2));
    P.v = make_rsrc(A.v + st * kDV, static_cast<uint32_t>(A.T) * (kDV * 2));
    P.ig = make_rsrc(A.ipre + st, static_cast<uint32_t>(A.T) * 4);
    P.fg = make_rsrc(A.fpre + st, static_cast<uint32_t>(A.T) * 4);
    const auto rdh = make_rsrc(A.dh + st * kDV, static_cast<uint32_t>(A.T) * (kDV * 2));
    const auto rq = make_rsrc(A.q + st * kDQK, static_cast<uint32_t>(A.T) * (kDQK * 2));
    const auto rX = make_rsrc(A.X + st * kDQK, static_cast<uint32_t>(A.T) * (kDQK * 4));
    const auto rqx = make_rsrc(A.qx + st * kPart, static_cast<uint32_t>(A.T) * (kPart * 4));
    const auto rn = make_rsrc(A.nst + static_cast<int64_t>(s) * A.NC * kDQK, static_cast<uint32_t>(A.NC) * (kDQK * 4));
    const auto rm = make_rsrc(A.mst + static_cast<int64_t>(s) * A.NC, static_cast<uint32_t>(A.NC) * 4);

    DState C;
    const float* nin;
    float m_prev;
    if (g == 0) {
        const float* C0 = A.C0 ? A.C0 + static_cast<int64_t>(s) * kCV : nullptr;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int pp = 0; pp < 4; ++pp)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    C[dt][pp][e] = C0 ? *reinterpret_cast<const f32x4_t*>(C0 + dtile_c0(d0, dt, vq, pp, e, lane)) : f32x4_t{};
        nin = A.n0 ? A.n0 + static_cast<int64_t>(s) * kDQK : nullptr;
        m_prev = A.m0 ? A.m0[s] : 0.0f;
    } else {
        MLSTM_CHECK(g * A.R - 1 >= 0 && g * A.R - 1 < A.NS, kDbgChunkBwd);
        const float* slot = A.seg + (static_cast<int64_t>(s) * A.NS + g * A.R - 1) * kSlotFloats;
        dtile_from_slot(C, slot, d0, vq, lane);
        nin = slot + kCV;
        m_prev = slot[kCV + kDQK + 2];
    }
    // element `lane` of this d tile's normaliser, the same in every wave
    float n = nin ? nin[kDTile * tile + lane] : 0.0f;
    float s_off = 0.0f;   // C = C_acc e^{s_off}
    float g_m = m_prev, g_s = 0.0f;
    float gi = 0.f, gf = 0.f;

    u32x4_t rdhv[8], rv[8], rk;
    u32x2_t rqv[2];   // q of the tau tile this wave finishes
    auto load = [&](int t0, int tid) {
        const int lane = tid & 63, krow = tid >> 3, kcol = 8 * (tid & 7);   // this thread's piece of the K tile
        rk = bload128(P.k, static_cast<uint32_t>(t0 + krow) * (kDQK * 2) + (kDTile * tile + kcol) * 2, 0);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
            rqv[dt] = bload64(rq, (static_cast<uint32_t>(t0 + 16 * vq + (lane & 15)) * kDQK + d0 + 16 * dt + 4 * (lane >> 4)) * 2);
    };
    if (c_begin < c_end) {
        const int t0 = c_begin * kBL;
        load_gates(gi, gf, P, t0, lane);
        load(t0, tid);
        load_rows512(rdhv, rdh, t0, tid);
        load_pieces<8>(rv, P.v, kDV * 2, t0, wave, lane);
        if (gate_wave) gate_phase(S.G[c_begin & 1], gi, gf, g_m, g_s, lane, A.T - t0);
        load_gates(gi, gf, P, t0 + kBL, lane);   // gates are loaded a chunk before their phase
    }
    const int tid_outer = tid;
    for (int c = c_begin; c < c_end; ++c) {
        MLSTM_OPAQUE_LANES(tid_outer);
        const int t0 = c * kBL;
        const GateBuf<true>& Gc = S.G[c & 1];
        __syncthreads();   // the previous chunk's readers are done; this chunk's gates are visible
        store_rows512(S.dH, rdhv, tid);
        store_transposed<8>(S.Vt, rv, wave, lane);
        float npart;   // this wave's eight rows of sum_t w_t k_t, columns 8 (lane % 8) + rows8_col of the tile
        {
            const int krow = tid >> 3, kcol = 8 * (tid & 7);
            const float w = Gc.wC[krow], wn = Gc.wb[krow];
            u32x4_t hi, lo;
            float kn[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float a = lo_f32(rk[i]) * w, b = hi_f32(rk[i]) * w;
                hi[i] = pack_bf16x2(a, b);
                lo[i] = pack_bf16x2(a - lo_f32(hi[i]), b - hi_f32(hi[i]));
                kn[2 * i] = lo_f32(rk[i]) * wn;
                kn[2 * i + 1] = hi_f32(rk[i]) * wn;
            }
            npart = rows8_sum(kn, lane);
            uint16_t* p0 = &S.Kw[0][krow * KP + kcol];   // 8-byte aligned rows
            uint16_t* p1 = &S.Kw[1][krow * KP + kcol];
            *reinterpret_cast<u32x2_t*>(p0) = u32x2_t{hi[0], hi[1]};
            *reinterpret_cast<u32x2_t*>(p0 + 4) = u32x2_t{hi[2], hi[3]};
            *reinterpret_cast<u32x2_t*>(p1) = u32x2_t{lo[0], lo[1]};
            *reinterpret_cast<u32x2_t*>(p1 + 4) = u32x2_t{lo[2], lo[3]};
        }
        const u32x2_t qv[2] = {rqv[0], rqv[1]};
        const int tn = min(c + 1, c_end - 1) * kBL;
        load(tn, tid);
        // n and m entering the chunk
        MLSTM_CHECK(c < A.NC, kDbgChunkBwd);
        bstoref(rn, tid < kDTile ? static_cast<uint32_t>(c * kDQK + kDTile * tile + tid) * 4u : kNoStore, n);
        bstoref(rm, tile == 0 && tid == 0 ? static_cast<uint32_t>(c) * 4u : kNoStore, m_prev);
        __syncthreads();   // the chunk's operands are visible
        // gates of the next chunk, one chunk ahead
        if (gate_wave && c + 1 < c_end) gate_phase(S.G[(c + 1) & 1], gi, gf, g_m, g_s, lane, A.T - (t0 + kBL));
        load_gates(gi, gf, P, t0 + 2 * kBL, lane);

        f32x4_t X[2][4];
        dtile_product<true>(X, C, S.dH, vq, lane, [&](int pp) {
            rdhv[2 * pp] = load_row512(rdh, tn, 2 * pp, tid);
            rdhv[2 * pp + 1] = load_row512(rdh, tn, 2 * pp + 1, tid);
        });
        const float esc = expf(s_off);
        const float decay_n = Gc.scal[0], m_next = Gc.scal[1], s_new = Gc.scal[2];
        const float c_scale = Gc.scal[3];   // != 1: apply this chunk's decay to C_acc eagerly
        __syncthreads();   // the dH rows are read; the exchange takes their place
        f32x4_t* ex = reinterpret_cast<f32x4_t*>(S.dH);
        dtile_give(ex, X, wave, lane);
        if (c_scale != 1.0f) {
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int pp = 0; pp < 4; ++pp)
#pragma unroll
                    for (int e = 0; e < 2; ++e) C[dt][pp][e] *= c_scale;
        }
        float* np = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(S.dH) + kExBytes);
        np[wave * kDTile + 8 * (lane & 7) + rows8_col(lane)] = npart;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            u32x4_t b[2][2];   // hi, lo
#pragma unroll
            for (int p = 0; p < 2; ++p)
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) b[p][dt] = tr_op(S.Kw[p], KP, 32 * ks, 32 * dp + 16 * dt, lane);
            dtile_update<2>(C, S.Vt, b, vq, ks, lane,
                            [&](int i) { rv[i] = load_piece<8>(P.v, kDV * 2, tn, i, wave, lane); });
            dtile_update_order<8, 8>();
        }
        __syncthreads();   // the exchange and the partial sums of n are visible
        float nsum = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) nsum += np[w * kDTile + lane];
        n = decay_n * n + nsum;
        f32x4_t Y[2];
        dtile_take(Y, ex, X, vq, dp, lane);
        const int tau = 16 * vq + l16;
        float qx = 0.0f;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
            Y[dt] *= esc;
            bstore128(rX, (static_cast<uint32_t>(t0 + tau) * kDQK + d0 + 16 * dt + 4 * g16) * 4u, Y[dt]);
            qx += dot4(qv[dt], Y[dt]);
        }
        qx = sum_rows4(qx) * kQScale;
        bstoref(rqx, g16 == 0 ? (static_cast<uint32_t>(t0 + tau) * kPart + 2 * tile + dp) * 4u : kNoStore, qx);
        s_off = s_new;
        m_prev = m_next;
    }
}

// ---- intra pass --------------------------------------------------------------------------------
// One workgroup of four waves per chunk, two workgroups per CU.  A wave owns 16 tau rows of every
// [tau][sigma] tile and of dq, so nothing but the staged K rows crosses waves: one barrier.  Q, V and dH
// come from memory in the operand layout (their rows are contiguous in the contraction index): staging them
// in LDS cost the second workgroup of a CU.
struct IntraSmem {
    uint16_t K[kBL * kQP];
    uint16_t tile[4][3][16 * kPP];   // per wave: St / den, P hi, P lo as [tau][sigma]
    float n[kDQK];
    float x[kBL], M[kBL], g[kBL], fl[kBL];
    int R[kBL];
};
static_assert(2 * sizeof(IntraSmem) <= 160 * 1024, "LDS budget for two workgroups per CU");

template <bool kBf16>
__global__ void __launch_bounds__(256, 2) bwd_intra_kernel(BwdParams A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    IntraSmem& S = *reinterpret_cast<IntraSmem*>(smem_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g16 = lane >> 4, l16 = lane & 15;
    const int c = blockIdx.x % A.NC, s = blockIdx.x / A.NC;
    const int T = A.T, t0 = c * kBL;
    // the tau block of this wave; its causal tiles number tw + 1, so every second chunk hands them out in
    // reverse and a SIMD gets light and heavy waves
    const int tw = (c & 1) ? 3 - wave : wave;
    const int64_t st = static_cast<int64_t>(s) * T, sc = static_cast<int64_t>(s) * A.NC + c;
    const auto rq = make_rsrc(A.q + st * kDQK, static_cast<uint32_t>(T) * kDQK * 2);
    const auto rk = make_rsrc(A.k + st * kDQK, static_cast<uint32_t>(T) * kDQK * 2);
    const auto rv = make_rsrc(A.v + st * kDV, static_cast<uint32_t>(T) * kDV * 2);
    const auto rdh = make_rsrc(A.dh + st * kDV, static_cast<uint32_t>(T) * kDV * 2);
    const auto rdq = grad_rsrc<kBf16>(A.dq, st, T, kDQK);
    const int tau = 16 * tw + l16;
    const bool valid = t0 + tau < T;

    u32x4_t kr[8], qf[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int e = tid + 256 * i;
        kr[i] = bload128(rk, static_cast<uint32_t>(t0 + (e >> 5)) * (kDQK * 2) + 16 * (e & 31), 0);
    }
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
        qf[ks] = bload128(rq, static_cast<uint32_t>(t0 + tau) * (kDQK * 2) + (32 * ks + 8 * g16) * 2, 0);
    S.n[tid] = A.nst[sc * kDQK + tid];
    if (wave == 0) {
        BGate G;
        float decay;
        bwd_gates(make_rsrc(A.ipre + st, static_cast<uint32_t>(T) * 4), make_rsrc(A.fpre + st, static_cast<uint32_t>(T) * 4),
                  T, t0, A.mst[sc], lane, G, decay);
        S.x[lane] = G.x;
        S.M[lane] = G.M;
        S.R[lane] = G.R;
        S.g[lane] = G.g;
        S.fl[lane] = G.fl;
        A.wk[sc * kBL + lane] = G.wk;
        if (lane == 0) A.decay[sc] = decay;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int e = tid + 256 * i;
        *reinterpret_cast<u32x4_t*>(&S.K[(e >> 5) * kQP + 8 * (e & 31)]) = kr[i];
    }
    __syncthreads();

    // S^T tiles of this wave: columns tau, rows sigma = 16 j + 4 g16 + 0..3 (j <= tw)
    f32x4_t Sa[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        Sa[j] = f32x4_t{};
        if (j <= tw)
#pragma unroll
            for (int ks = 0; ks < 8; ++ks) Sa[j] = mfma16(row_op(S.K, kQP, 16 * j, 32 * ks, lane), qf[ks], Sa[j]);
    }
    const float Mt = S.M[tau];
    const int Rt = S.R[tau];
    const float gt = S.g[tau];
    const float flt = S.fl[tau];
    float Et[4][4];
    float rsum = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int sg = 16 * j + 4 * g16 + r;
            const float xs = S.x[sg];
            const float e = (sg <= tau && sg >= Rt && xs != -INFINITY) ? fexp(xs - Mt) : 0.0f;
            Et[j][r] = e;
            Sa[j][r] = Sa[j][r] * kQScale * e;
            rsum += Sa[j][r];
        }
    rsum = sum_rows4(rsum);
    float qn = 0.0f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
        for (int e = 0; e < 8; ++e) qn += bf_at(qf[ks], e) * S.n[32 * ks + 8 * g16 + e];
    qn = sum_rows4(qn) * kQScale;
    const float Dt = gt * qn + rsum;
    const float den = fmaxf(fabsf(Dt), flt);
    const bool act = fabsf(Dt) > flt;
    // a row past the end has D = 0, and a floor that underflows once m exceeds 87: its 1 / den would be inf, and
    // inf * 0 would enter the products over tau
    const float rden = valid ? 1.0f / den : 0.0f;
    const float gd = gt * rden;
    uint16_t* tSn = S.tile[wave][0];
    uint16_t* tPh = S.tile[wave][1];
    uint16_t* tPl = S.tile[wave][2];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        *reinterpret_cast<u32x2_t*>(&tSn[l16 * kPP + 16 * j + 4 * g16]) =
            u32x2_t{pack_bf16x2(Sa[j][0] * rden, Sa[j][1] * rden), pack_bf16x2(Sa[j][2] * rden, Sa[j][3] * rden)};

    // (V dH^T) on the same tiles, both operands from memory, four k steps of loads together
    f32x4_t Ap[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) Ap[j] = f32x4_t{};
#pragma unroll 1
    for (int k4 = 0; k4 < 4; ++k4) {
        u32x4_t hb[4], va[4][4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t col = static_cast<uint32_t>(32 * (4 * k4 + u) + 8 * g16) * 2;
            hb[u] = bload128(rdh, static_cast<uint32_t>(t0 + tau) * (kDV * 2) + col, 0);
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (j <= tw) va[j][u] = bload128(rv, static_cast<uint32_t>(t0 + 16 * j + l16) * (kDV * 2) + col, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (j <= tw)
#pragma unroll
                for (int u = 0; u < 4; ++u) Ap[j] = mfma16(va[j][u], hb[u], Ap[j]);
    }
    // the first half of this wave's rows of X and q for dq (the stores of dq may alias X as far as the
    // compiler knows, so the loads of a half are issued together here)
    f32x4_t x[8];
    u32x2_t qv[8];
    const int64_t row = (st + t0 + tau) * kDQK + 4 * g16;
    auto load_x = [&](int half) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            x[i] = f32x4_t{};
            qv[i] = u32x2_t{0u, 0u};
            if (valid) {
                x[i] = *reinterpret_cast<const f32x4_t*>(A.X + row + 16 * (8 * half + i));
                qv[i] = *reinterpret_cast<const u32x2_t*>(A.q + row + 16 * (8 * half + i));
            }
        }
    };
    load_x(0);
    // dh_t . N_t from its two parts: the entry state's g q^_t . X_t and the intra
    // sum_sigma St_t,sigma (dh_t . v_sigma); then w_t
    float dhn = 0.0f;
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) dhn += Sa[j][r] * Ap[j][r];
    dhn = sum_rows4(dhn);
    if (valid) {
        const f32x4_t* pp = reinterpret_cast<const f32x4_t*>(&A.qx[(st + t0 + tau) * kPart]);
        const f32x4_t p = pp[0] + pp[1];
        dhn += gt * ((p[0] + p[1]) + (p[2] + p[3]));
    }
    const float wt = (act && valid) ? -(dhn * rden) * (Dt > 0.0f ? 1.0f : -1.0f) * rden : 0.0f;
    const float gwt = gt * wt;
    if (g16 == 0) {
        A.gd[sc * kBL + tau] = gd * kQScale;
        A.gw[sc * kBL + tau] = gwt * kQScale;
    }
    // P^T [sigma][tau] = E o (A'^T / den + w), kept as P [tau][sigma] in bf16 hi + lo: where the
    // numerator and denominator terms of a row nearly cancel, P's own rounding would show
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float pv[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) pv[r] = Et[j][r] * (Ap[j][r] * rden + wt);
        const uint32_t h01 = pack_bf16x2(pv[0], pv[1]), h23 = pack_bf16x2(pv[2], pv[3]);
        *reinterpret_cast<u32x2_t*>(&tPh[l16 * kPP + 16 * j + 4 * g16]) = u32x2_t{h01, h23};
        *reinterpret_cast<u32x2_t*>(&tPl[l16 * kPP + 16 * j + 4 * g16]) =
            u32x2_t{pack_bf16x2(pv[0] - lo_f32(h01), pv[1] - hi_f32(h01)),
                    pack_bf16x2(pv[2] - lo_f32(h23), pv[3] - hi_f32(h23))};
    }
    // the tiles transposed to [sigma][tau] for the reverse walks, whose B operands they are (a wave's own
    // LDS accesses stay in order; the clobber keeps the compiler from moving reads of other lanes' writes)
    asm volatile("" ::: "memory");
    {
        uint16_t* oS = A.SnT + sc * (kBL * kBL);
        uint16_t* oP = A.PT + sc * (2 * kBL * kBL);
        const int src = (4 * g16 + (l16 >> 2)) * kPP + 4 * (l16 & 3);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int dst = (16 * j + l16) * kBL + 16 * tw + 4 * g16;
            *reinterpret_cast<u32x2_t*>(oS + dst) = tr_read(&tSn[src + 16 * j]);
            *reinterpret_cast<u32x2_t*>(oP + dst) = tr_read(&tPh[src + 16 * j]);
            *reinterpret_cast<u32x2_t*>(oP + kBL * kBL + dst) = tr_read(&tPl[src + 16 * j]);
        }
    }
    // dq^T [d][tau] = (g / den X + sum_sigma K^T[d][sigma] P^T[sigma][tau] + g w n) / sqrt(DQK);
    // r_t = q_t . dq_t
    u32x4_t ph[2], pl[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        ph[ks] = row_op(tPh, kPP, 0, 32 * ks, lane);
        pl[ks] = row_op(tPl, kPP, 0, 32 * ks, lane);
    }
    float rr = 0.0f;
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        f32x4_t o[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int db = 8 * half + i;
            f32x4_t acc = f32x4_t{};
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                if (ks <= tw / 2) {
                    const u32x4_t a = tr_op(S.K, kQP, 32 * ks, 16 * db, lane);
                    acc = mfma16(a, ph[ks], acc);
                    acc = mfma16(a, pl[ks], acc);
                }
#pragma unroll
            for (int r = 0; r < 4; ++r) o[i][r] = (gd * x[i][r] + acc[r] + gwt * S.n[16 * db + 4 * g16 + r]) * kQScale;
            rr += dot4(qv[i], o[i]);
        }
        if (half == 0) load_x(1);
#pragma unroll
        for (int i = 0; i < 8; ++i)   // rows past the end are dropped
            store_grad<kBf16>(rdq, static_cast<uint32_t>(t0 + tau) * kDQK + 4 * g16 + 16 * (8 * half + i), o[i]);
    }
    rr = sum_rows4(rr);
    if (valid && g16 == 0) A.r[st + t0 + tau] = rr;
}

// ---- reverse combine ----------------------------------------------------------------------------
// Running gradients of the segment exits from the local ones, in place: slot j (time order over the
// segments 1..G-1, R sub-segments each) receives the gradient of the state entering sub-segment j from
// everything at or after it; slot g R is then what reaches the exit of segment g.
__global__ void __launch_bounds__(256) bwd_rev_combine_kernel(float* seg, int NS, int R) {
    constexpr int kE4 = static_cast<int>(kCV + kDQK) / 4;
    const int e4 = blockIdx.x * 256 + threadIdx.x;
    if (e4 >= kE4) return;
    float* base = seg + static_cast<int64_t>(blockIdx.y) * NS * kSlotFloats;
    f32x4_t cur = f32x4_t{};
    constexpr int kBatch = 8;   // slots whose loads are issued together
    for (int j1 = NS - 1; j1 >= 0; j1 -= kBatch) {
        f32x4_t loc[kBatch];
        float dec[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (j1 - u >= 0) {
                const float* slot = base + static_cast<int64_t>(j1 - u) * kSlotFloats;
                loc[u] = reinterpret_cast<const f32x4_t*>(slot)[e4];
                dec[u] = slot[kCV + kDQK + 1];
            }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (j1 - u >= 0) {
#pragma unroll
                for (int r = 0; r < 4; ++r) cur[r] = dec[u] * cur[r] + loc[u][r];
                if ((j1 - u) % R == 0) reinterpret_cast<f32x4_t*>(base + static_cast<int64_t>(j1 - u) * kSlotFloats)[e4] = cur;
            }
    }
}

// ---- dk: reverse walk over a 64-row tile of d -----------------------------------------------------
// Per chunk, last to first, with Gam_c (the gradient reaching the chunk's exit) in registers:
//   dk^T[d][sigma] = wk_sigma (sum_v Gam[d][v] V[sigma][v] + gam[d]) + sum_tau Q^T[d][tau] P[tau][sigma] / sqrt(DQK)
//   Gam <- decay Gam + Q^T (g / den / sqrt(DQK) dH),   gam <- decay gam + Q^T (g w / sqrt(DQK))
// The weight g / den goes on Q, rounded once to bf16: dk sums Gam over v, so a rounding of a q element stays
// a relative one of each term, where one of dH would be relative to dH's length in the product dH . V, which
// is far smaller (the dv walk, which sums over d, puts it on dH for the same reason: on Q its largest row
// error was 2.7 times as large).  Gam enters its product as a bf16 pair: c = k . dk and the reverse sums of r - c are
// taken from the unrounded dk, and with Gam rounded once di~ was off by 7.5e-4 of its norm (5.3e-4 with the pair) and
// df~ by 1.0e-2 (7.2e-3) at 1 x 2048 tokens; it costs 13 us of 760 at 16 x 4096.  gam's weights enter as three
// bf16 rows (24 bits).
struct DkSmem {
    uint16_t Ht[kDV * kTP];        // dH^T, rows in pair order
    uint16_t V[kBL * kRP];         // the chunk's V rows, then the exchange of the partial products
    uint16_t Q[2][kBL * kTP];      // the chunk's Q rows, this d tile's 64 columns: plain, times g / den / sqrt(DQK)
    float wk[kBL], gw[kBL];
    float gam[2][kDTile];
    float red[kWaves];
};
static_assert(sizeof(DkSmem) <= 160 * 1024, "LDS budget");

template <bool kBf16>
__global__ void __launch_bounds__(kThreads, 1) bwd_dk_kernel(BwdParams A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    DkSmem& S = *reinterpret_cast<DkSmem*>(smem_raw);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int dp = wave & 1, vq = wave >> 1;
    const int wi = work_index();
    const int tile = wi % kNDT;
    const int g = (wi / kNDT) % A.G;
    const int s = wi / kNDT / A.G;
    const int d0 = kDTile * tile + 32 * dp;
    const int c_begin = g * A.seg_chunks;
    const int c_end = min(A.NC, c_begin + A.seg_chunks);
    MLSTM_CHECK(s < A.S, kDbgChunkBwd);
    const int64_t st = static_cast<int64_t>(s) * A.T;
    const auto rq = make_rsrc(A.q + st * kDQK, static_cast<uint32_t>(A.T) * (kDQK * 2));
    const auto rv = make_rsrc(A.v + st * kDV, static_cast<uint32_t>(A.T) * (kDV * 2));
    const auto rdh = make_rsrc(A.dh + st * kDV, static_cast<uint32_t>(A.T) * (kDV * 2));
    const auto rk = make_rsrc(A.k + st * kDQK, static_cast<uint32_t>(A.T) * (kDQK * 2));
    const auto rdk = grad_rsrc<kBf16>(A.dk, st, A.T, kDQK);
    const auto rc = make_rsrc(A.kdk + st * kPart, static_cast<uint32_t>(A.T) * (kPart * 4));

    DState Gm;
    if (g < A.G - 1) {
        MLSTM_CHECK(g * A.R < A.NS, kDbgChunkBwd);
        const float* slot = A.seg + (static_cast<int64_t>(s) * A.NS + g * A.R) * kSlotFloats;
        dtile_from_slot(Gm, slot, d0, vq, lane);
        if (tid < kDTile) S.gam[0][tid] = slot[kCV + kDTile * tile + tid];
    } else {   // nothing reaches the last chunk's exit state
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int pp = 0; pp < 4; ++pp) Gm[dt][pp][0] = Gm[dt][pp][1] = f32x4_t{};
        if (tid < kDTile) S.gam[0][tid] = 0.0f;
    }

    u32x4_t rvv[8], rh[8], rqv;
    float rgd;
    float rwk = 0.0f, rgw = 0.0f, rdec = 1.0f;
    auto load = [&](int c, int tid) {
        const int lane = tid & 63, qrow = tid >> 3, qcol = 8 * (tid & 7);
        const int t0 = c * kBL;
        const int64_t sc = (static_cast<int64_t>(s) * A.NC + c) * kBL;
        rqv = bload128(rq, static_cast<uint32_t>(t0 + qrow) * (kDQK * 2) + (kDTile * tile + qcol) * 2, 0);
        rgd = A.gd[sc + qrow];
        rwk = A.wk[sc + lane];
        rgw = A.gw[sc + lane];
        rdec = A.decay[static_cast<int64_t>(s) * A.NC + c];
    };
    if (c_begin < c_end) {
        load(c_end - 1, tid);
        load_rows512(rvv, rv, (c_end - 1) * kBL, tid);
        load_pieces<8>(rh, rdh, kDV * 2, (c_end - 1) * kBL, wave, lane);
    }

    int par = 0;
    const int tid_outer = tid;
    for (int c = c_end - 1; c >= c_begin; --c, par ^= 1) {
        MLSTM_OPAQUE_LANES(tid_outer);
        const int t0 = c * kBL;
        const int64_t sc = static_cast<int64_t>(s) * A.NC + c;
        __syncthreads();   // the previous chunk's readers are done; gam is visible
        store_transposed<8>(S.Ht, rh, wave, lane);
        store_rows512(S.V, rvv, tid);
        *reinterpret_cast<u32x4_t*>(&S.Q[0][(tid >> 3) * kTP + 8 * (tid & 7)]) = rqv;
        *reinterpret_cast<u32x4_t*>(&S.Q[1][(tid >> 3) * kTP + 8 * (tid & 7)]) = scale8(rqv, rgd);
        S.wk[lane] = rwk;   // every wave the same values
        S.gw[lane] = rgw;
        const float decay = rdec;
        // P^T and k of the sigma tile this wave finishes (requested before the next chunk's loads: memory
        // answers in order)
        const int sg = 16 * vq + l16;
        u32x4_t ph[2], pl[2];
        u32x2_t kv[2];
        {
            const uint16_t* p = A.PT + sc * (2 * kBL * kBL) + sg * kBL + 8 * g16;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                ph[ks] = lds16(p + 32 * ks);
                pl[ks] = lds16(p + kBL * kBL + 32 * ks);
            }
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
                kv[dt] = bload64(rk, (static_cast<uint32_t>(t0 + sg) * kDQK + d0 + 16 * dt + 4 * g16) * 2u);
        }
        const int tn = max(c - 1, c_begin) * kBL;
        load(max(c - 1, c_begin), tid);
        __syncthreads();   // the chunk's operands are visible
        f32x4_t X[2][4];
        dtile_product<true>(X, Gm, S.V, vq, lane, [&](int pp) {
            rh[2 * pp] = load_piece<8>(rdh, kDV * 2, tn, 2 * pp, wave, lane);
            rh[2 * pp + 1] = load_piece<8>(rdh, kDV * 2, tn, 2 * pp + 1, wave, lane);
        });
        __syncthreads();   // the V rows are read; the exchange takes their place
        f32x4_t* ex = reinterpret_cast<f32x4_t*>(S.V);
        dtile_give(ex, X, wave, lane);

#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
#pragma unroll
            for (int pp = 0; pp < 4; ++pp)
#pragma unroll
                for (int e = 0; e < 2; ++e) Gm[dt][pp][e] *= decay;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            u32x4_t bw[1][2];   // the weighted Q read transposed: columns d of this wave, k = tau
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) bw[0][dt] = tr_op(S.Q[1], kTP, 32 * ks, 32 * dp + 16 * dt, lane);
            dtile_update<1>(Gm, S.Ht, bw, vq, ks, lane,
                            [&](int i) { rvv[i] = load_row512(rv, tn, i, tid); });
            dtile_update_order<4, 4>();
        }
        u32x4_t b[2][2];   // [ks][dt]: plain Q, the same way
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) b[ks][dt] = tr_op(S.Q[0], kTP, 32 * ks, 32 * dp + 16 * dt, lane);
        if (vq == 0) {
            f32x4_t zacc[2] = {f32x4_t{}, f32x4_t{}};
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                u32x4_t wa = u32x4_t{0u, 0u, 0u, 0u};
                if (l16 < 3) {   // rows 0, 1, 2: the weights' leading, second and third bf16 parts
                    float w[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        w[e] = S.gw[32 * ks + 8 * g16 + e];
                        const float a = bf16_to_f32(f32_to_bf16(w[e]));
                        if (l16 > 0) w[e] -= a;
                        const float a2 = bf16_to_f32(f32_to_bf16(w[e]));
                        if (l16 > 1) w[e] -= a2;
                    }
#pragma unroll
                    for (int e = 0; e < 4; ++e) wa[e] = pack_bf16x2(w[2 * e], w[2 * e + 1]);
                }
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) zacc[dt] = mfma16(wa, b[ks][dt], zacc[dt]);
            }
            if (g16 == 0) {
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) {
                    const int d = 32 * dp + 16 * dt + l16;
                    S.gam[par ^ 1][d] = decay * S.gam[par][d] + (zacc[dt][0] + (zacc[dt][1] + zacc[dt][2]));
                }
            }
        }
        // the intra term on this wave's sigma tile (P is zero for tau < sigma)
        f32x4_t in[2] = {f32x4_t{}, f32x4_t{}};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
            if (32 * ks + 31 >= 16 * vq)
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) {
                    in[dt] = mfma16(b[ks][dt], ph[ks], in[dt]);
                    in[dt] = mfma16(b[ks][dt], pl[ks], in[dt]);
                }
        const float w = S.wk[sg];
        f32x4_t gam[2];
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) gam[dt] = *reinterpret_cast<const f32x4_t*>(&S.gam[par][32 * dp + 16 * dt + 4 * g16]);
        __syncthreads();   // the exchange is visible
        f32x4_t Y[2];
        dtile_take(Y, ex, X, vq, dp, lane);
        float cp = 0.0f;
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
            f32x4_t o;
#pragma unroll
            for (int r = 0; r < 4; ++r) o[r] = w * (Y[dt][r] + gam[dt][r]) + kQScale * in[dt][r];
            store_grad<kBf16>(rdk, static_cast<uint32_t>(t0 + sg) * kDQK + d0 + 16 * dt + 4 * g16, o);
            cp += dot4(kv[dt], o);
        }
        cp = sum_rows4(cp);
        bstoref(rc, g16 == 0 ? (static_cast<uint32_t>(t0 + sg) * kPart + 2 * tile + dp) * 4u : kNoStore, cp);
    }
    if (A.dC0 == nullptr || g != 0) return;
    // Gam_{-1}, gam_{-1}: the gradients of C0 and n0, and this tile's share of dm0
    __syncthreads();
    float dm = 0.0f;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int pp = 0; pp < 4; ++pp)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int64_t o = static_cast<int64_t>(s) * kCV + dtile_c0(d0, dt, vq, pp, e, lane);
                *reinterpret_cast<f32x4_t*>(A.dC0 + o) = Gm[dt][pp][e];
                if (A.C0) {
                    const f32x4_t c0 = *reinterpret_cast<const f32x4_t*>(A.C0 + o);
                    const f32x4_t& x = Gm[dt][pp][e];
                    dm += (x[0] * c0[0] + x[1] * c0[1]) + (x[2] * c0[2] + x[3] * c0[3]);
                }
            }
    if (tid < kDTile) {
        const int64_t o = static_cast<int64_t>(s) * kDQK + kDTile * tile + tid;
        const float x = S.gam[par][tid];
        A.dn0[o] = x;
        if (A.n0) dm += x * A.n0[o];
    }
    dm = wave_total(dm);
    if (lane == 0) S.red[wave] = dm;
    __syncthreads();
    if (tid == 0) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) t += S.red[w];
        A.dmp[s * kNDT + tile] = t;
    }
}

// ---- dv: reverse walk over a 128-column tile of v --------------------------------------------------
// Wave w = 2 vq + dh owns the 128 x 32 block d = 128 dh + 0..127, v = 128 tile + 32 vq + 0..31 of Gam as
// tiles (vt, pp, e): lane (l16, g16) holds Gam[d = 128 dh + 32 pp + 8 g16 + 4 e + j][v = 32 vq + 16 vt + l16],
// the A operand of dv^T[v][sigma] = sum_d Gam[d][v] K[sigma][d] with 16-byte reads of K rows.  The two
// halves of d meet in LDS (the wave of half dh finishes the sigma tiles 2 dh and 2 dh + 1; X[vt][i] is the
// sigma tile (2 dh + i) % 4).  Per chunk,
// last to first:
//   dv^T[v][sigma] = wk_sigma (sum_d Gam[d][v] K[sigma][d]) + sum_tau dH^T[v][tau] (St / den)[tau][sigma]
//   Gam <- decay Gam + Q^T (g / den / sqrt(DQK) dH)
// with the scaled dH rounded once to bf16 (see the dk walk).
constexpr int kKP = kDQK + 16;   // pitch of the K rows (544 bytes)
constexpr int kHP = kDVT + 8;    // pitch of the dH rows (272 bytes)
struct DvSmem {
    uint16_t Qt[kDQK * kTP];     // Q^T, rows in pair order
    uint16_t K[kBL * kKP];
    uint16_t dH[2][kBL * kHP];   // the chunk's dH rows, this tile's 128 columns: plain, times g / den / sqrt(DQK)
    f32x4_t ex[kWaves][4][64];   // partial products handed to the other half of d
    float wk[kBL];
};
static_assert(sizeof(DvSmem) <= 160 * 1024, "LDS budget");

template <bool kBf16>
__global__ void __launch_bounds__(kThreads, 1) bwd_dv_kernel(BwdParams A) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    DvSmem& S = *reinterpret_cast<DvSmem*>(smem_raw);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g16 = lane >> 4, l16 = lane & 15;
    const int dh = wave & 1, vq = wave >> 1;
    const int wi = work_index();
    const int tile = wi % kNTile;
    const int g = (wi / kNTile) % A.G;
    const int s = wi / kNTile / A.G;
    const int v0 = kDVT * tile;
    const int c_begin = g * A.seg_chunks;
    const int c_end = min(A.NC, c_begin + A.seg_chunks);
    MLSTM_CHECK(s < A.S, kDbgChunkBwd);
    const int64_t st = static_cast<int64_t>(s) * A.T;
    const auto rq = make_rsrc(A.q + st * kDQK, static_cast<uint32_t>(A.T) * (kDQK * 2));
    const auto rk = make_rsrc(A.k + st * kDQK, static_cast<uint32_t>(A.T) * (kDQK * 2));
    const auto rdh = make_rsrc(A.dh + st * kDV, static_cast<uint32_t>(A.T) * (kDV * 2));
    const auto rdv = grad_rsrc<kBf16>(A.dv, st, A.T, kDV);

    f32x4_t Gm[2][4][2];
    if (g < A.G - 1) {
        MLSTM_CHECK(g * A.R < A.NS, kDbgChunkBwd);
        const float* slot = A.seg + (static_cast<int64_t>(s) * A.NS + g * A.R) * kSlotFloats;
#pragma unroll
        for (int vt = 0; vt < 2; ++vt)
#pragma unroll
            for (int pp = 0; pp < 4; ++pp)
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    Gm[vt][pp][e] = *reinterpret_cast<const f32x4_t*>(
                        slot + slot_c4(32 * dh + 8 * pp + 2 * g16 + e, v0 + 32 * vq + 16 * vt + l16));
    } else {
#pragma unroll
        for (int vt = 0; vt < 2; ++vt)
#pragma unroll
            for (int pp = 0; pp < 4; ++pp) Gm[vt][pp][0] = Gm[vt][pp][1] = f32x4_t{};
    }

    u32x4_t rkv[4], rqv[4], rhv[2];
    float rgd[2];
    float rwk = 0.0f, rdec = 1.0f;
    auto load = [&](int c) {
        const int t0 = c * kBL;
        const int64_t sc = (static_cast<int64_t>(s) * A.NC + c) * kBL;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            rhv[i] = bload128(rdh, static_cast<uint32_t>(t0 + (tid >> 4) + 32 * i) * (kDV * 2) + (v0 + 8 * (tid & 15)) * 2, 0);
#pragma unroll
        for (int i = 0; i < 2; ++i) rgd[i] = A.gd[sc + (tid >> 4) + 32 * i];
        rwk = A.wk[sc + lane];
        rdec = A.decay[static_cast<int64_t>(s) * A.NC + c];
    };
    auto load_k = [&](int t0, int i) {
        rkv[i] = bload128(rk, static_cast<uint32_t>(t0 + (tid >> 5) + 16 * i) * (kDQK * 2) + 16 * (tid & 31), 0);
    };
    if (c_begin < c_end) {
        load(c_end - 1);
#pragma unroll
        for (int i = 0; i < 4; ++i) load_k((c_end - 1) * kBL, i);
        load_pieces<4>(rqv, rq, kDQK * 2, (c_end - 1) * kBL, wave, lane);
    }

    for (int c = c_end - 1; c >= c_begin; --c) {
        const int t0 = c * kBL;
        const int64_t sc = static_cast<int64_t>(s) * A.NC + c;
        __syncthreads();   // the previous chunk's readers are done
#pragma unroll
        for (int i = 0; i < 4; ++i)
            *reinterpret_cast<u32x4_t*>(&S.K[((tid >> 5) + 16 * i) * kKP + 8 * (tid & 31)]) = rkv[i];
        store_transposed<4>(S.Qt, rqv, wave, lane);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int off = ((tid >> 4) + 32 * i) * kHP + 8 * (tid & 15);
            *reinterpret_cast<u32x4_t*>(&S.dH[0][off]) = rhv[i];
            *reinterpret_cast<u32x4_t*>(&S.dH[1][off]) = scale8(rhv[i], rgd[i]);
        }
        S.wk[lane] = rwk;   // every wave the same values
        const float decay = rdec;
        // (St / den)^T of the two sigma tiles this wave finishes
        u32x4_t sn[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                sn[i][ks] = lds16(A.SnT + sc * (kBL * kBL) + (16 * (2 * dh + i) + l16) * kBL + 32 * ks + 8 * g16);
        const int tn = max(c - 1, c_begin) * kBL;
        load(max(c - 1, c_begin));
        __syncthreads();   // the chunk's operands are visible

        f32x4_t X[2][4];
#pragma unroll
        for (int vt = 0; vt < 2; ++vt)
#pragma unroll
            for (int tb = 0; tb < 4; ++tb) X[vt][tb] = f32x4_t{};
#pragma unroll
        for (int pp = 0; pp < 4; ++pp) {
            u32x4_t b[4];
#pragma unroll
            for (int tb = 0; tb < 4; ++tb) b[tb] = row_op(S.K, kKP, 16 * ((2 * dh + tb) & 3), 128 * dh + 32 * pp, lane);
            load_k(tn, pp);
#pragma unroll
            for (int vt = 0; vt < 2; ++vt) {
                const u32x4_t a = pack8(Gm[vt][pp][0], Gm[vt][pp][1]);
#pragma unroll
                for (int tb = 0; tb < 4; ++tb) X[vt][tb] = mfma16(a, b[tb], X[vt][tb]);
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int vt = 0; vt < 2; ++vt) S.ex[wave][2 * i + vt][lane] = X[vt][2 + i];

#pragma unroll
        for (int vt = 0; vt < 2; ++vt)
#pragma unroll
            for (int pp = 0; pp < 4; ++pp)
#pragma unroll
                for (int e = 0; e < 2; ++e) Gm[vt][pp][e] *= decay;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            u32x4_t hw[2];   // the weighted dH read transposed: columns v of this wave, k = tau
#pragma unroll
            for (int vt = 0; vt < 2; ++vt) hw[vt] = tr_op(S.dH[1], kHP, 32 * ks, 32 * vq + 16 * vt, lane);
#pragma unroll
            for (int pp = 0; pp < 4; ++pp) {
                if (pp & 1) rqv[2 * ks + pp / 2] = load_piece<4>(rq, kDQK * 2, tn, 2 * ks + pp / 2, wave, lane);
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const u32x4_t a = row_op(S.Qt, kTP, 128 * dh + 32 * pp + 16 * e, 32 * ks, lane);
#pragma unroll
                    for (int vt = 0; vt < 2; ++vt) Gm[vt][pp][e] = mfma16(a, hw[vt], Gm[vt][pp][e]);
                }
            }
        }
        u32x4_t hb[2][2];   // plain dH, the same way
#pragma unroll
        for (int vt = 0; vt < 2; ++vt)
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) hb[vt][ks] = tr_op(S.dH[0], kHP, 32 * ks, 32 * vq + 16 * vt, lane);
        // the intra term on this wave's sigma tiles (St is zero for tau < sigma)
        f32x4_t in[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int vt = 0; vt < 2; ++vt) {
                in[i][vt] = f32x4_t{};
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
                    if (ks >= dh) in[i][vt] = mfma16(hb[vt][ks], sn[i][ks], in[i][vt]);
            }
        __syncthreads();   // the exchange is visible
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int sg = 16 * (2 * dh + i) + l16;
            // rows past the end are dropped, all as row T: T may be up to 2^21 - 1, and the byte offset of an fp32
            // row 2^21 is 2^32
            const uint32_t row = static_cast<uint32_t>(min(t0 + sg, A.T));
            const float w = S.wk[sg];
#pragma unroll
            for (int vt = 0; vt < 2; ++vt) {
                const f32x4_t y = X[vt][i] + S.ex[wave ^ 1][2 * i + vt][lane];
                store_grad<kBf16>(rdv, row * kDV + v0 + 32 * vq + 16 * vt + 4 * g16, w * y + in[i][vt]);
            }
        }
    }
}

// ---- gate gradients ----------------------------------------------------------------------------
constexpr int kGT = 1024;   // threads of the gate pass: one block of kGT tokens per step of its scan
__global__ void __launch_bounds__(kGT) bwd_gate_kernel(BwdParams A) {
    const int s = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int T = A.T;
    const int64_t st = static_cast<int64_t>(s) * T;
    __shared__ float wsum[kGT / 64];
    double carry = 0.0;
    for (int base = ((T + kGT - 1) / kGT - 1) * kGT; base >= 0; base -= kGT) {
        const int t = base + tid;
        float val = 0.0f, ci = 0.0f;
        if (t < T) {
            const f32x4_t* p = reinterpret_cast<const f32x4_t*>(&A.kdk[(st + t) * kPart]);
            const f32x4_t p2 = p[0] + p[1];
            ci = (p2[0] + p2[1]) + (p2[2] + p2[3]);
            val = A.r[st + t] - ci;
        }
        // inclusive prefix over the block, then the suffix sum from t on
        const float incl = wave_incl_sum(val);
        __syncthreads();   // wsum of the previous block is consumed
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        float before = 0.0f, total = 0.0f;
#pragma unroll
        for (int w = 0; w < kGT / 64; ++w) {
            if (w < wave) before += wsum[w];
            total += wsum[w];
        }
        const float suffix = total - (before + incl) + val;
        if (t < T) {
            const float f = A.fpre[st + t];
            const double da = carry + static_cast<double>(suffix);
            A.dfp[st + t] = (f == -INFINITY) ? 0.0f : static_cast<float>(da / (1.0 + exp(static_cast<double>(f))));
            A.dip[st + t] = ci;
        }
        carry += static_cast<double>(total);
    }
    if (A.dm0 && tid == 0) {
        float dm = 0.0f;
#pragma unroll
        for (int b = 0; b < kNDT; ++b) dm += A.dmp[s * kNDT + b];
        A.dm0[s] = dm;
    }
}

// T = 0: the initial-state gradients are zero
__global__ void __launch_bounds__(256) bwd_zero_state_kernel(float* dC0, float* dn0, float* dm0, int S) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (i < static_cast<int64_t>(S) * kCV) dC0[i] = 0.0f;
    if (i < static_cast<int64_t>(S) * kDQK) dn0[i] = 0.0f;
    if (i < S) dm0[i] = 0.0f;
}

template <class Smem, bool kBf16>
hipError_t launch_pass(void (*kern)(BwdParams), const BwdParams& p, unsigned grid, int threads, hipStream_t stream) {
    static std::atomic<uint64_t> raised{0};   // one per kernel: every pass has an LDS layout of its own
    hipError_t e = raise_dynamic_lds(reinterpret_cast<const void*>(kern), sizeof(Smem), raised);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), sizeof(Smem), stream, p);
    return hipGetLastError();
}

size_t align256(size_t b) { return (b + 255) & ~static_cast<size_t>(255); }

// The workspace size callers are told (mlstm_chunkwise_bwd_workspace_bytes), a fixed formula of the
// interface: per sequence and chunk but the first a state slot and a bf16 state matrix, the segment slots,
// four fp32 copies of q, and per-token terms.  The passes below use about an eighth of it (94 KB of 1 MB per
// chunk, and the segment slots).
size_t published_workspace_bytes(int64_t S, int T) {
    const int64_t NC = (T + kBL - 1) / kBL, NC1 = NC > 0 ? NC - 1 : 0;
    return align256(static_cast<size_t>(S * NC1 * kSlotFloats) * 4) +
           align256(chunk_mfma_workspace_bytes(static_cast<int>(S), 1, T, kDQK, kDV, kBL)) +
           align256(static_cast<size_t>(4 * S * T * kDQK) * 4) + align256(static_cast<size_t>(S * NC1 * kCV) * 2) +
           align256(static_cast<size_t>(S * (kCV + kDQK)) * 4) + align256(static_cast<size_t>(S * NC * kDQK) * 4) +
           align256(static_cast<size_t>(S * T) * 4) + align256(static_cast<size_t>(S * T * 8) * 4) +
           align256(static_cast<size_t>(S * NC) * 4) + align256(static_cast<size_t>(S * 129) * 4);
}

// Lays the arrays of the passes out in the workspace; returns the bytes used.  A chunk of 64 tokens
// takes 64 KB of X, 24 KB of St and P and about 6 KB of scalars and states, under the 256 KB of the four
// copies of q that the published size counts for a full chunk; what rounding a partial chunk up to 64
// tokens adds is under the 513 KB it counts once per sequence.
size_t lay_out(BwdParams& p, unsigned char* ws) {
    const int64_t S = p.S, T = p.T, NC = p.NC;
    size_t off = 0;
    auto take = [&](int64_t bytes) {
        unsigned char* at = ws + off;
        off += align256(static_cast<size_t>(bytes));
        return at;
    };
    p.seg = reinterpret_cast<float*>(take(S * p.NS * kSlotFloats * 4));
    p.X = reinterpret_cast<float*>(take(S * T * kDQK * 4));
    p.nst = reinterpret_cast<float*>(take(S * NC * kDQK * 4));
    p.mst = reinterpret_cast<float*>(take(S * NC * 4));
    p.decay = reinterpret_cast<float*>(take(S * NC * 4));
    p.wk = reinterpret_cast<float*>(take(S * NC * kBL * 4));
    p.gd = reinterpret_cast<float*>(take(S * NC * kBL * 4));
    p.gw = reinterpret_cast<float*>(take(S * NC * kBL * 4));
    p.SnT = reinterpret_cast<uint16_t*>(take(S * NC * kBL * kBL * 2));
    p.PT = reinterpret_cast<uint16_t*>(take(S * NC * kBL * kBL * 4));
    p.qx = reinterpret_cast<float*>(take(S * T * kPart * 4));
    p.kdk = reinterpret_cast<float*>(take(S * T * kPart * 4));
    p.r = reinterpret_cast<float*>(take(S * T * 4));
    p.dmp = reinterpret_cast<float*>(take(S * kNDT * 4));
    return off;
}

}  // namespace

bool chunk_bwd_supported(mlstm_dtype dt, int DQK, int DV, int L) {
    return dt == MLSTM_BF16 && DQK == kDQK && DV == kDV && L == kBL;
}

size_t chunk_bwd_workspace_bytes(int B, int NH, int T) {
    return published_workspace_bytes(static_cast<int64_t>(B) * NH, T);
}

hipError_t launch_chunk_bwd(const ChunkBwdArgs& a, void* workspace, hipStream_t stream) {
    const int S = a.f.B * a.f.NH, T = a.f.T;
    if (S == 0) return hipSuccess;
    if (T == 0) {
        if (a.dC0) {
            const int64_t n = static_cast<int64_t>(S) * kCV;
            hipLaunchKernelGGL(bwd_zero_state_kernel, dim3(static_cast<unsigned>((n + 255) / 256)), dim3(256), 0, stream,
                               a.dC0, a.dn0, a.dm0, S);
            return hipGetLastError();
        }
        return hipSuccess;
    }
    BwdParams p{};
    p.q = static_cast<const uint16_t*>(a.f.q);
    p.k = static_cast<const uint16_t*>(a.f.k);
    p.v = static_cast<const uint16_t*>(a.f.v);
    p.dh = static_cast<const uint16_t*>(a.dh);
    p.ipre = a.f.ipre;
    p.fpre = a.f.fpre;
    p.C0 = a.f.C0;
    p.n0 = a.f.n0;
    p.m0 = a.f.m0;
    p.dq = a.dq;
    p.dk = a.dk;
    p.dv = a.dv;
    p.dip = a.dipre;
    p.dfp = a.dfpre;
    p.dC0 = a.dC0;
    p.dn0 = a.dn0;
    p.dm0 = a.dm0;
    p.S = S;
    p.T = T;
    p.NC = (T + kBL - 1) / kBL;
    const SegmentShape sh = segment_shape(a.f.B, a.f.NH, T, kBL, true);
    p.G = sh.G;
    p.R = sh.R;
    p.NS = (sh.G - 1) * sh.R;
    p.seg_chunks = sh.seg_chunks;
    if (lay_out(p, static_cast<unsigned char*>(workspace)) > published_workspace_bytes(S, T)) return hipErrorInvalidValue;

    hipError_t e = launch_segment_states(a.f, kBL, sh, p.seg, true, stream);
    if (e != hipSuccess) return e;
    const unsigned walks = static_cast<unsigned>(S) * p.G * kNDT;
    e = launch_pass<XSmem, false>(bwd_x_kernel, p, walks, kThreads, stream);
    if (e != hipSuccess) return e;
    e = a.grads_bf16 ? launch_pass<IntraSmem, true>(bwd_intra_kernel<true>, p, static_cast<unsigned>(S) * p.NC, 256, stream)
                     : launch_pass<IntraSmem, false>(bwd_intra_kernel<false>, p, static_cast<unsigned>(S) * p.NC, 256, stream);
    if (e != hipSuccess) return e;
    if (p.G > 1) {   // the forward's segment slots are consumed: the gradients take their place
        const ReverseLocal rl{p.q, p.dh, p.gd, p.gw, p.decay, p.seg, S, T, p.NC, p.NS, p.R, p.seg_chunks};
        e = launch_reverse_local(rl, stream);
        if (e != hipSuccess) return e;
        constexpr int kE4 = static_cast<int>(kCV + kDQK) / 4;
        hipLaunchKernelGGL(bwd_rev_combine_kernel, dim3((kE4 + 255) / 256, S), dim3(256), 0, stream, p.seg, p.NS, p.R);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    e = a.grads_bf16 ? launch_pass<DkSmem, true>(bwd_dk_kernel<true>, p, walks, kThreads, stream)
                     : launch_pass<DkSmem, false>(bwd_dk_kernel<false>, p, walks, kThreads, stream);
    if (e != hipSuccess) return e;
    e = a.grads_bf16 ? launch_pass<DvSmem, true>(bwd_dv_kernel<true>, p, walks, kThreads, stream)
                     : launch_pass<DvSmem, false>(bwd_dv_kernel<false>, p, walks, kThreads, stream);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(bwd_gate_kernel, dim3(S), dim3(kGT), 0, stream, p);
    return hipGetLastError();
}

#ifdef MLSTM_DEBUG
MLSTM_DEBUG_READER(debug_flags_chunk_bwd)
#endif

}  // namespace mlstm

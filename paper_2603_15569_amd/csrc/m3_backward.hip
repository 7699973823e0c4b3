// Backward pass of the chunked prefill scan (training; Sec. 3.3 "Chunked
// Algorithm for MIMO SSMs": the same chunk decomposition run in reverse) on
// gfx950, bf16 inputs, N = 128, P = 64, chunks of 64 rows (chunk * rank =
// 64: SISO chunk 64, rank 2 chunk 32, rank 4 chunk 16).
//
// Forward, per chunk c with chunk-local prefix sums cum_t (of dt A) and
// psi_t (of theta), C^_t = R(-psi_t) C_t, B^_j = R(-psi_j) B_j, gamma_t =
// lambda_t dt_t, sigma_j = gamma_j + (1 - lambda_{j+1}) dt_{j+1},
// w_tt = gamma_t, w_tj = e^{cum_t - cum_j} sigma_j (j < t), v_j = e^{cum_e -
// cum_j} sigma_j (e the chunk's last token):
//   y_t = sum_{j<=t} w_tj (C^_t . B^_j) x_j + e^{cum_t} C^_t^T S_{c-1} + D x_t
//   S_c = R(psi_e) (e^{cum_e} S_{c-1} + M_c),  M_c = sum_j v_j B^_j x_j^T
// Reverse, for a loss J with dy = dJ/dy and G_c = dJ/dS_c (G_last = dJ/d
// final state):
//   U_c = R(-psi_e) G_c                                  (dJ/dM_c)
//   G_{c-1} = e^{cum_e} U_c + sum_t e^{cum_t} C^_t dy_t^T
//   dG[t][j] = dy_t . x_j (chunk rows), G[t][j] = C^_t . B^_j
//   dx_j  = sum_t w_tj G[t][j] dy_t + D dy_j + v_j U^T B^_j
//   dB^_j = sum_t w_tj dG[t][j] C^_t + v_j U x_j
//   dC^_t = sum_j w_tj dG[t][j] B^_j + e^{cum_t} S_{c-1} dy_t
//   dJ/dw_tj = dG[t][j] G[t][j] -> cum_t, cum_j, sigma_j (j < t), gamma_t (j = t)
//   dJ/dv_j = <B^_j, U x_j>      -> cum_e, cum_j, sigma_j
//   y's state term               -> cum_t (e^{cum_t} <C^_t, S_{c-1} dy_t>)
//   S_c's rotation and decay     -> psi_e, cum_e
//   dpsi_t[i] = (dC^ x C^ + dB^ x B^)_t[i] (the 2-D cross product of the
//   pair (i, i + N/2)), dB = R(psi_t) dB^, dC = R(psi_t) dC^;
//   then the prefix sums are transposed (suffix sums over the chunk:
//   d(dt_u A_u) = sum_{t>=u} dcum_t, dtheta_u = sum_{t>=u} dpsi_t) and the
//   chain runs through gamma, sigma, dt, lambda and A.
//
// A slice's chunks are split into segments (one or more per slice, so that
// the launch fills the device); one workgroup carries the state and its
// gradient through its segment in registers.  Kernels (one stream, in order):
//   k_bwd_aggr   per (segment, direction), only with several segments a
//                slice: the segment's map of the forward state (first to last
//                chunk) or of the state gradient (last to first), from zero,
//                with the sums of cum_e and psi_e                     (MFMA)
//   k_bwd_pass   per slice: the maps folded over the segments
//   k_bwd_main   per segment: a forward sweep that stores the state entering
//                each chunk (bf16), then the chunks last to first, each with
//                U from the carried gradient and every gradient of its tokens
//                                                                     (MFMA)
//   k_bwd_finish per-head sums of dA and dD (fixed order); the sigma term
//                that crosses a segment boundary
// Bound: the bytes (per 64-row chunk 96 KB of inputs and gradients, 28 KB of
// B and x read again by the forward sweep, 32 KB of bf16 states written and
// read) and, with two waves a SIMD, the latencies of k_bwd_main's dependent
// steps.  One fp32 map of the state per chunk and direction, written by a
// kernel over all chunks and folded by a second one, moved 352 KB a chunk and
// took 8.62 ms on B=8 L=4096 H=32 rank 4 and 313 us on B=4 L=2048 H=16 SISO;
// carrying the state through a segment in registers takes 2.65 ms and 157 us.
// Operands are bf16 with fp32 accumulation (as the forward); the carried
// state and gradient, the prefix sums, weights and every scalar gradient are
// fp32.  Results are deterministic: no atomics.
#include <stddef.h>

#include <algorithm>

#include "m3_device.h"
#include "m3_internal.h"
#include "m3_scan_common.h"

namespace m3 {
namespace {

using namespace scan;

constexpr int kN = 128, kP = 64, kNH = 64, kRows = 64;
constexpr int kNW = 8, kThr = kNW * kWave;
constexpr int LDN = kN + 16;  // bf16 row strides (32-byte padding: FShape::PAD)
constexpr int LDP = kP + 16;
constexpr int LDC = kNH + 4;  // cos / sin rows (as many dwords apart)
constexpr int kMap = kN * kP;
constexpr int kTot = 1 + 2 * kNH;   // a segment's totals: log-decay (base 2), cosines and sines of its angles
constexpr float kLog2e = 1.44269504088896340736f;
typedef Mma<bf16> MM;
// four floats at 4-byte alignment (the angles' arrays need no more)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Lane and wave coordinates of a 512-thread workgroup.  The carried N x P
// state is held transposed in MFMA tiles: wave (it, ph) owns the positions
// 16 it + l16 (q = 0) and 64 + 16 it + l16 (q = 1) of N and the positions
// 16 (2 ph + u) + 4 g + v of P, element st[q][u][v].  Positions are in tile
// order (chan_of) everywhere in LDS and registers: pair `i` of the lane is
// chan_of(16 it + l16).
struct Lane {
    int tid, lane, wave, g, l16, it, ph, i;
    __device__ __forceinline__ Lane() : Lane((int)threadIdx.x) {}
    __device__ __forceinline__ explicit Lane(int tid_) {
        tid = tid_;
        lane = tid & (kWave - 1);
        wave = __builtin_amdgcn_readfirstlane(tid / kWave);
        g = lane >> 4;
        l16 = lane & 15;
        it = wave & 3;
        ph = wave >> 2;
        i = chan_of(16 * it + l16);
    }
};
typedef f32x4 State[2][2];

// A chunk's scalars by row (token, rank): base-2 log-decay prefix, gamma,
// sigma, v, e^{cum}; its total log-decay and the pairs' total angles.
struct alignas(16) Tok {   // (read in 16-byte pieces, in every slot of an array)
    float c2[kRows], gam[kRows], sig[kRows], v[kRows], ec[kRows];
    float psie[kNH], ce[kNH], se[kNH];   // psi_e, its cosine and sine
    float c2e;
};
static_assert(offsetof(Tok, c2) % 16 == 0 && offsetof(Tok, sig) % 16 == 0, "16-byte pieces");

// Sums over the 16 lanes of a row group of the values of TT tokens (v[0 ..
// TT - 1] in every lane): the lane l16 < TT gets token l16's.  Four at once by
// a butterfly (11 operations and one masked store, against 16 and four).
template <int TT> __device__ __forceinline__ float sum16_each(const float (&v)[TT], int l16) {
    if constexpr (TT == 4) {
        const bool o1 = l16 & 1, o2 = l16 & 2;
        const float a = (o1 ? v[1] : v[0]) + dpp_src<0xB1, 0xf>(o1 ? v[0] : v[1]);
        const float b = (o1 ? v[3] : v[2]) + dpp_src<0xB1, 0xf>(o1 ? v[2] : v[3]);
        float r = (o2 ? b : a) + dpp_src<0x4E, 0xf>(o2 ? a : b);
        r += dpp_src<0x128, 0xf>(r);
        r += dpp_src<0x124, 0xf>(r);
        return r;
    } else if constexpr (TT == 2) {
        const bool o1 = l16 & 1;
        float r = (o1 ? v[1] : v[0]) + dpp_src<0xB1, 0xf>(o1 ? v[0] : v[1]);
        r += dpp_src<0x128, 0xf>(r);
        r += dpp_src<0x124, 0xf>(r);
        r += dpp_src<0x122, 0xf>(r);
        return r;
    } else {
        return sum16(v[0]);
    }
}
// Sum over the R lanes of a token's rank rows.
template <int R> __device__ __forceinline__ float sum_rank(float v) {
    if constexpr (R >= 2) v += dpp_src<0xB1, 0xf>(v);   // quad_perm: lane ^ 1
    if constexpr (R >= 4) v += dpp_src<0x4E, 0xf>(v);   // quad_perm: lane ^ 2
    return v;
}
// Inclusive suffix sums over the tokens of a 16-lane row group (R equal
// lanes a token).
template <int R> __device__ __forceinline__ float suffix16(float v) {
    if constexpr (R == 1) v += dpp_src<0x101, 0xf>(v);   // row_shl:1
    if constexpr (R <= 2) v += dpp_src<0x102, 0xf>(v);
    v += dpp_src<0x104, 0xf>(v);
    v += dpp_src<0x108, 0xf>(v);
    return v;
}
// ---------------------------------------------------------------------------
// Chunk prologue, in two steps with a barrier between them, each on values
// loaded a chunk earlier.
// ---------------------------------------------------------------------------
template <int R> struct Shp {
    static constexpr int Q = kRows / R;
    static constexpr int TPS = Q / kNW;   // tokens whose angles a thread scans
};

struct Slice {   // the slice's offsets
    int64_t b, h, tok;   // tok: (b L) H + h, the slice's first scalar
};

// Where a thread's loads stand in the chunk to be loaded next, as token indices
// (b L + t) H + h advanced a chunk at a time, so that no load needs a 64-bit
// product: `th` its first angle token, `row` its staged row's token.
struct Cur {
    int64_t th, row, t0;   // t0: the chunk's first token
};
// Steps back to the last valid token for a token t past the end (only the
// sequence's last chunk is ragged: a branch rarely taken).
__device__ __forceinline__ int64_t past_end(int t, int nvalid, int q, int64_t stride) {
    int64_t o = 0;
    if (nvalid < q) {
        asm volatile("");   // (a branch, not selects on every load)
        o = t >= nvalid ? (nvalid - 1 - t) * stride : 0;
    }
    return o;
}

// Raw values of a chunk's prologue: wave w's tokens w TPS .. of the angles
// (pair = lane), and, by wave 0 with one lane a row, the token's scalars.
template <int R>
struct RawTok {
    float th[Shp<R>::TPS];
    float dt, lam, A, dtn, lamn;
};

template <int R>
__device__ __forceinline__ void load_tok(const BwdArgs &a, const Slice &s, const Lane &w, const Cur &u, int nvalid,
                                         RawTok<R> &r) {
    constexpr int Q = Shp<R>::Q, TPS = Shp<R>::TPS;
#pragma unroll
    for (int k = 0; k < TPS; ++k)
        r.th[k] = a.theta[(u.th + k * a.H + past_end(w.wave * TPS + k, nvalid, Q, a.H)) * kNH + w.lane];
    if (w.wave == 0) {
        const int64_t t = u.t0 + min(w.lane / R, nvalid - 1), tn = min(t + 1, a.L - 1);
        r.dt = a.dt[s.tok + t * a.H];
        r.lam = a.lam[s.tok + t * a.H];
        r.A = a.A[s.b * a.a_sb + t * a.a_st + s.h * a.a_sh];
        r.dtn = a.dt[s.tok + tn * a.H];
        r.lamn = a.lam[s.tok + tn * a.H];
    }
}

// Step 1: each wave's angle prefix sums (its total to `seg`), and wave 0 the
// scalar tables.  Tokens past the end of the sequence get zero angles and
// weights.
template <int R>
__device__ __forceinline__ void tok_scan(const BwdArgs &a, const Lane &w, int64_t c, int nvalid, const RawTok<R> &r,
                                         float (&ps)[Shp<R>::TPS], float (*seg)[kNH], Tok &o) {
    constexpr int Q = Shp<R>::Q, TPS = Shp<R>::TPS;
#pragma unroll
    for (int k = 0; k < TPS; ++k) ps[k] = r.th[k];
    if (nvalid < Q) {
#pragma unroll
        for (int k = 0; k < TPS; ++k) ps[k] = w.wave * TPS + k < nvalid ? ps[k] : 0.f;
    }
#pragma unroll
    for (int k = 1; k < TPS; ++k) ps[k] += ps[k - 1];
    seg[w.wave][w.lane] = ps[TPS - 1];
    if (w.wave == 0) {
        const int t = w.lane / R;
        const bool in = t < nvalid;
        // (scaled before the sum, so that a prefix is rounded once)
        const float c2 = lane_scan(in && w.lane % R == 0 ? r.dt * r.A * kLog2e : 0.f);
        const float c2e = lane_bcast(c2, nvalid * R - 1);
        const float gam = in ? r.lam * r.dt : 0.f;
        float sig = gam;
        if (in && c * Q + t + 1 < a.L) sig += (1.f - r.lamn) * r.dtn;
        o.c2[w.lane] = c2;
        o.gam[w.lane] = gam;
        o.sig[w.lane] = sig;
        o.v[w.lane] = in ? exp2_fast(c2e - c2) * sig : 0.f;
        o.ec[w.lane] = in ? exp2_fast(c2) : 0.f;
        if (w.lane == 0) o.c2e = c2e;
    }
}

// Step 2: the cos / sin table of psi_t, and psi_e with its own in fp32.
template <int R>
__device__ __forceinline__ void tok_table(const Lane &w, int nvalid, const float (&ps)[Shp<R>::TPS],
                                          const float (*seg)[kNH], h2 *cs, Tok &o) {
    constexpr int TPS = Shp<R>::TPS;
    float off = 0.f;
    for (int s = 0; s < w.wave; ++s) off += seg[s][w.lane];
    float pe = 0.f, se = 0.f, ce = 0.f;
#pragma unroll
    for (int k = 0; k < TPS; ++k) {
        const float psi = ps[k] + off;
        float sn, cn;
        sincos_rev(psi, &sn, &cn);
        cs_put(&cs[(w.wave * TPS + k) * LDC + w.lane], cn, sn);
        if (k == (nvalid - 1) % TPS) {
            pe = psi;
            se = sn;
            ce = cn;
        }
    }
    if (w.wave == (nvalid - 1) / TPS) {
        o.psie[w.lane] = pe;
        o.ce[w.lane] = ce;
        o.se[w.lane] = se;
    }
}

// ---------------------------------------------------------------------------
// Row staging: one thread a (row, 16-byte piece).
// ---------------------------------------------------------------------------
struct RowAt {   // this thread's task
    int row, cp, t, r;
};
template <int R> __device__ __forceinline__ RowAt row_at(const Lane &w) {
    RowAt k;
    k.row = w.tid / 8;
    k.cp = w.tid % 8;
    k.t = k.row / R;
    k.r = k.row % R;
    return k;
}
// B or C piece pair (channels i and i + N/2) of the thread's row at token `at`.
struct Pair { bf16x8 lo, hi; };
template <int R>
__device__ __forceinline__ Pair load_pair(const RowAt &k, const void *src, int64_t at) {
    const bf16 *p = static_cast<const bf16 *>(src) + (at * R + k.r) * kN + k.cp * 8;
    return Pair{*reinterpret_cast<const bf16x8 *>(p), *reinterpret_cast<const bf16x8 *>(p + kNH)};
}
template <int R>
__device__ __forceinline__ bf16x8 load_row(const RowAt &k, const void *src, int64_t at) {
    return *reinterpret_cast<const bf16x8 *>(static_cast<const bf16 *>(src) + (at * R + k.r) * kP + k.cp * 8);
}
// Rotated by -psi_t (cos c, sin s of the thread's eight pairs) into [row][LDN].
__device__ __forceinline__ void put_rot(bf16 *dst, const RowAt &k, const Pair &v, const float (&c)[8],
                                        const float (&s)[8]) {
    Pair o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float u = (float)v.lo[e], x = (float)v.hi[e];
        o.lo[e] = (bf16)(c[e] * u + s[e] * x);
        o.hi[e] = (bf16)(c[e] * x - s[e] * u);
    }
    put_tile_order(&dst[k.row * LDN], k.cp, o.lo);
    put_tile_order(&dst[k.row * LDN + kNH], k.cp, o.hi);
}
__device__ __forceinline__ void put_scaled(bf16 *dst, const RowAt &k, bf16x8 v, float sc) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (bf16)(sc * (float)v[e]);
    put_tile_order(&dst[k.row * LDP], k.cp, v);
}

// ---------------------------------------------------------------------------
// State in registers
// ---------------------------------------------------------------------------
// S <- R(sgn psi) S on the lane's pair, and S <- f S.
__device__ __forceinline__ void rotate(State &st, float cn, float sn) {
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float re = st[0][u][v], im = st[1][u][v];
            st[0][u][v] = cn * re - sn * im;
            st[1][u][v] = sn * re + cn * im;
        }
}
__device__ __forceinline__ void scale(State &st, float f) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < 2; ++u) st[q][u] *= f;
}
__device__ __forceinline__ void zero(State &st) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < 2; ++u) st[q][u] = f32x4{0.f, 0.f, 0.f, 0.f};
}
// st += rows^T (N x K) scaled-rows (K x P): K = the chunk's 64 rows.
__device__ __forceinline__ void add_outer(State &st, const bf16 *rows, const bf16 *cols, const Lane &w) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        bf16x8 pc[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) pc[u] = load_kt(cols, LDP, ks * 32, (2 * w.ph + u) * 16, w.g, w.l16);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const bf16x8 nr = load_kt(rows, LDN, ks * 32, (4 * q + w.it) * 16, w.g, w.l16);
#pragma unroll
            for (int u = 0; u < 2; ++u) st[q][u] = MM::mma(pc[u], nr, st[q][u]);
        }
    }
}
// fp32 maps: the API's [n][p] arrays, and the workspace's (in thread order).
__device__ __forceinline__ void load_np(State &st, const float *m, const Lane &w) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            st[q][u] = *reinterpret_cast<const f32x4 *>(
                &m[(64 * q + w.i) * kP + 32 * w.ph + 8 * w.g + 4 * u]);
}
__device__ __forceinline__ void store_np(const State &st, float *m, const Lane &w) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            *reinterpret_cast<f32x4 *>(
                &m[(64 * q + w.i) * kP + 32 * w.ph + 8 * w.g + 4 * u]) = st[q][u];
}
__device__ __forceinline__ void load_map(State &st, const float *m, const Lane &w) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            st[q][u] = *reinterpret_cast<const f32x4 *>(&m[(2 * q + u) * 4 * kThr + 4 * w.tid]);
}
__device__ __forceinline__ void store_map(const State &st, float *m, const Lane &w) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            *reinterpret_cast<f32x4 *>(&m[(2 * q + u) * 4 * kThr + 4 * w.tid]) = st[q][u];
}
// The state entering a chunk, bf16 in thread order (each thread reads back
// what it wrote).
struct SBf { bf16x8 q[2]; };   // q: [u][v]
__device__ __forceinline__ SBf to_bf(const State &st) {
    SBf o;
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int v = 0; v < 4; ++v) o.q[q][4 * u + v] = (bf16)st[q][u][v];
    return o;
}
__device__ __forceinline__ void store_sbf(bf16 *m, const SBf &o, const Lane &w) {
    *reinterpret_cast<bf16x8 *>(&m[8 * w.tid]) = o.q[0];
    *reinterpret_cast<bf16x8 *>(&m[8 * (kThr + w.tid)]) = o.q[1];
}
__device__ __forceinline__ SBf load_sbf(const bf16 *m, const Lane &w) {
    return SBf{{*reinterpret_cast<const bf16x8 *>(&m[8 * w.tid]),
                *reinterpret_cast<const bf16x8 *>(&m[8 * (kThr + w.tid)])}};
}

// ---------------------------------------------------------------------------
// Sweep of the carried state over n chunks: forward (kFwd) from chunk c0 up,
//   S <- R(psi_e) (e^{cum_e} S + sum_j v_j B^_j x_j^T),
// or of its gradient from chunk c0 down,
//   G <- e^{cum_e} R(-psi_e) G + sum_t e^{cum_t} C^_t dy_t^T.
// With Sst, the state entering each chunk is stored (and one more after the
// last: n + 1 stores when n covers all but the segment's last chunk).
// Returns the sums of cum_e (base 2) and of the lane's psi_e (in fp64: thousands
// of radians in a long segment).  Two barriers a
// chunk; the next chunk's rows and the prologue values of the one after are in
// flight while a chunk is worked on.
// ---------------------------------------------------------------------------
template <int R> struct SweepLds {
    bf16 rows[kRows * LDN], cols[kRows * LDP];
    h2 cs[Shp<R>::Q * LDC];
    float seg[kNW][kNH];
    Tok tok[3];
};

template <int R, bool kFwd>
__device__ __forceinline__ void sweep(const BwdArgs &a, const Slice &s, const Lane &w, SweepLds<R> &L, int64_t c0,
                                      int64_t n, State &st, bf16 *Sst, double *sum_c2, double *sum_psi) {
    constexpr int Q = Shp<R>::Q, TPS = Shp<R>::TPS;
    constexpr int kDir = kFwd ? 1 : -1;
    const void *rsrc = kFwd ? a.B : a.C, *csrc = kFwd ? a.x : a.dy;
    const RowAt ra = row_at<R>(w);
    const int64_t ce = c0 + kDir * (n - 1);   // the last chunk
    auto valid = [&](int64_t c) { return (int)min((int64_t)Q, a.L - c * Q); };
    auto next = [&](int64_t c) { return c == ce ? c : c + kDir; };   // (past the last: loaded unused)
    Cur u;
    u.t0 = c0 * Q;
    u.th = s.tok + (u.t0 + w.wave * TPS) * a.H;
    u.row = s.tok + (u.t0 + ra.t) * a.H;
    RawTok<R> raw;
    float ps[TPS];
    Pair pr;
    bf16x8 px;
    auto fetch = [&](int64_t c) {
        const int64_t at = u.row + past_end(ra.t, valid(c), Q, a.H);
        pr = load_pair<R>(ra, rsrc, at);
        px = load_row<R>(ra, csrc, at);
        u.row += c == ce ? 0 : kDir * Q * a.H;
    };
    auto fetch_tok = [&](int64_t c) {
        load_tok<R>(a, s, w, u, valid(c), raw);
        u.th += c == ce ? 0 : kDir * Q * a.H;
        u.t0 += c == ce ? 0 : kDir * Q;
    };
    auto stage = [&](int nv, const Tok &o) {
        const bool in = ra.t < nv;
        float c[8], sn[8];
        cs_getn<8>(&L.cs[ra.t * LDC + ra.cp * 8], c, sn);
        if (nv < Q) {   // rows past the end are zero
            const bf16x8 z = {};
            if (!in) pr.lo = pr.hi = px = z;
        }
        put_rot(L.rows, ra, pr, c, sn);
        put_scaled(L.cols, ra, px, kFwd ? o.v[ra.row] : o.ec[ra.row]);
    };
    *sum_c2 = 0.0;
    *sum_psi = 0.0;
    int p0 = 0, p1 = 1, p2 = 2;   // scalar tables of this chunk, the next, the one after
    if (n > 0) {
        const int64_t c1 = next(c0), c2 = next(c1);
        fetch_tok(c0);
        fetch(c0);
        tok_scan<R>(a, w, c0, valid(c0), raw, ps, L.seg, L.tok[p0]);
        fetch_tok(c1);
        __syncthreads();
        tok_table<R>(w, valid(c0), ps, L.seg, L.cs, L.tok[p0]);
        __syncthreads();
        stage(valid(c0), L.tok[p0]);
        fetch(c1);
        tok_scan<R>(a, w, c1, valid(c1), raw, ps, L.seg, L.tok[p1]);
        fetch_tok(c2);
        __syncthreads();
    }
    int64_t c = c0;
    for (int64_t k = 0; k < n; ++k) {
        const int64_t c1 = next(c), c2 = next(c1), c3 = next(c2);
        // (a) this chunk's state update; the next one's table
        {
            const Tok &o = L.tok[p0];
            if (Sst) store_sbf(Sst + c * kMap, to_bf(st), w);
            const float e = exp2_fast(o.c2e), cn = o.ce[w.i], sn = o.se[w.i];
            *sum_c2 += o.c2e;
            *sum_psi += o.psie[w.i];
            if constexpr (!kFwd) rotate(st, cn, -sn);
            scale(st, e);
            add_outer(st, L.rows, L.cols, w);
            if constexpr (kFwd) rotate(st, cn, sn);
        }
        tok_table<R>(w, valid(c1), ps, L.seg, L.cs, L.tok[p1]);
        __syncthreads();
        // (b) the next chunk's rows; the scans of the one after
        stage(valid(c1), L.tok[p1]);
        fetch(c2);
        tok_scan<R>(a, w, c2, valid(c2), raw, ps, L.seg, L.tok[p2]);
        fetch_tok(c3);
        const int p = p0;
        p0 = p1;
        p1 = p2;
        p2 = p;
        c += kDir;
        __syncthreads();
    }
    if (Sst) store_sbf(Sst + c * kMap, to_bf(st), w);
}

__device__ __forceinline__ Slice slice_of(const BwdArgs &a, int64_t bh) {
    Slice s;
    s.b = bh / a.H;
    s.h = bh % a.H;
    s.tok = s.b * a.L * a.H + s.h;
    return s;
}

// ---------------------------------------------------------------------------
// k_bwd_aggr: grid (slices, segments - 1, 2): the forward map of segment y,
// or the gradient map of segment y + 1.
// ---------------------------------------------------------------------------
template <int R>
__global__ __launch_bounds__(kThr, 4) void k_bwd_aggr(BwdArgs a) {
    __shared__ __attribute__((aligned(16))) SweepLds<R> L;
    const Lane w;
    const int64_t bh = blockIdx.x;
    const Slice s = slice_of(a, bh);
    const bool fwd = blockIdx.z == 0;
    const int64_t seg = blockIdx.y + (fwd ? 0 : 1);
    const int64_t c0 = seg * a.G, n = min(a.G, a.nchunks - c0);
    State st;
    zero(st);
    double sc, sp;
    if (fwd) sweep<R, true>(a, s, w, L, c0, n, st, nullptr, &sc, &sp);
    else sweep<R, false>(a, s, w, L, c0 + n - 1, n, st, nullptr, &sc, &sp);
    const int64_t slot = bh * a.nseg + seg;
    store_map(st, (fwd ? a.Af : a.Ar) + slot * kMap, w);
    float *tot = a.tot + (slot * 2 + (fwd ? 0 : 1)) * kTot;
    if (w.ph == 0 && w.g == 0) {
        float sn, cn;
        sincos_sum(sp, &sn, &cn);
        tot[1 + w.i] = cn;
        tot[1 + kNH + w.i] = sn;
    }
    if (w.tid == 0) tot[0] = (float)sc;
}

// ---------------------------------------------------------------------------
// k_bwd_pass: grid (slices, 2, 2): the fold over a slice's segments, forward
// or reverse (z), of the tile columns u = y; the folded maps replace the
// segments' own (Af[s]: the state after segment s, from init_state; Ar[s]:
// the gradient of the state entering segment s, from dfinal).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kThr) void k_bwd_pass(BwdArgs a) {
    const Lane w;
    const int64_t bh = blockIdx.x;
    const int u = blockIdx.y;
    const bool fwd = blockIdx.z == 0;
    const float *src = fwd ? a.init_state : a.dfinal;
    f32x4 re = {0.f, 0.f, 0.f, 0.f}, im = re;
    if (src) {
        const float *m = src + bh * kMap + 32 * w.ph + 8 * w.g + 4 * u;
        re = *reinterpret_cast<const f32x4 *>(&m[w.i * kP]);
        im = *reinterpret_cast<const f32x4 *>(&m[(64 + w.i) * kP]);
    }
    float *M = fwd ? a.Af : a.Ar;
    const int n = (int)a.nseg - 1;
    constexpr int DEPTH = 4;   // segments whose loads are issued together
    for (int k0 = 0; k0 < n; k0 += DEPTH) {
        f32x4 mr[DEPTH], mi[DEPTH];
        float c2[DEPTH], cs[DEPTH], ss[DEPTH];
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int k = min(k0 + d, n - 1);
            const int64_t slot = bh * a.nseg + (fwd ? k : a.nseg - 1 - k);
            const float *tot = a.tot + (slot * 2 + (fwd ? 0 : 1)) * kTot;
            c2[d] = tot[0];
            cs[d] = tot[1 + w.i];
            ss[d] = tot[1 + kNH + w.i];
            const float *m = M + slot * kMap + 4 * w.tid;
            mr[d] = *reinterpret_cast<const f32x4 *>(&m[u * 4 * kThr]);
            mi[d] = *reinterpret_cast<const f32x4 *>(&m[(2 + u) * 4 * kThr]);
        }
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            if (k0 + d >= n) break;
            const int64_t slot = bh * a.nseg + (fwd ? k0 + d : a.nseg - 1 - (k0 + d));
            const float e = exp2_fast(c2[d]), cn = cs[d], sn = fwd ? ss[d] : -ss[d];
            f32x4 nr, ni;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                nr[v] = e * (cn * re[v] - sn * im[v]) + mr[d][v];
                ni[v] = e * (sn * re[v] + cn * im[v]) + mi[d][v];
            }
            re = nr;
            im = ni;
            float *m = M + slot * kMap + 4 * w.tid;
            *reinterpret_cast<f32x4 *>(&m[u * 4 * kThr]) = re;
            *reinterpret_cast<f32x4 *>(&m[(2 + u) * 4 * kThr]) = im;
        }
    }
}

// ---------------------------------------------------------------------------
// k_bwd_main: one workgroup a segment (grid: slices x segments).  After the
// forward sweep, the chunks last to first.  Wave (J, hf) owns row tile J of
// the chunk as columns j (dx, dB^) and as rows t (dC^), for the half hf of
// the columns p and of the rotation pairs.  Every output tile is formed
// transposed, from operands in tile order, so a lane holds eight consecutive
// channels of one row: 16-byte stores, the row's weights are per-lane scalars,
// and the sums over a row are in-lane.
// ---------------------------------------------------------------------------
template <int R> struct MainLds {
    bf16 B[kRows * LDN], C[kRows * LDN];
    bf16 X[kRows * LDP], Y[kRows * LDP], EY[kRows * LDP];   // x, dy, e^{cum} dy
    bf16 S[kN * LDP], U[kN * LDP];                          // S_{c-1}, U_c  [n][p]
    h2 cs[2][Shp<R>::Q * LDC];
    Tok tok[2];
    float seg[kNW][kNH];
    float rc[4][kRows], rg[kRows];     // sums of the mask terms by token row group
    float cc[kRows], csg[kRows];       // by column: cum, sigma
    float dv[2][kRows], dcy[2][kRows]; // dJ/dv_j and the y state term of cum_t, by half
    alignas(16) float dps[2][kNH];     // state terms of psi_e (by column half)
    alignas(16) float dth[4][kNH];     // dpsi totals of the row tiles
    float dcm[kNW];                    // state term of cum_e
    float red[kNW];
};

template <int R>
__global__ __launch_bounds__(kThr, 2) void k_bwd_main(BwdArgs a) {
    constexpr int Q = Shp<R>::Q;
    constexpr int TT = 4 / R;   // tokens among a lane's four accumulator rows
    __shared__ __attribute__((aligned(16))) char mem[std::max(sizeof(SweepLds<R>), sizeof(MainLds<R>))];
    SweepLds<R> &SW = *reinterpret_cast<SweepLds<R> *>(mem);
    MainLds<R> &M = *reinterpret_cast<MainLds<R> *>(mem);
    static_assert(offsetof(SweepLds<R>, cs) % 16 == 0 && offsetof(MainLds<R>, cs) % 16 == 0 &&
                      offsetof(MainLds<R>, S) % 16 == 0 && sizeof(MainLds<R>) <= 160 * 1024,
                  "16-byte pieces; a compute unit's LDS");
    Lane w;
    const int64_t bh = blockIdx.x, seg = blockIdx.y;
    const Slice s = slice_of(a, bh);
    const int64_t cb = seg * a.G, n = min(a.G, a.nchunks - cb), slot = bh * a.nseg + seg;
    const bool last = seg == a.nseg - 1;
    bf16 *Sst = static_cast<bf16 *>(a.Sst) + bh * a.nchunks * kMap;
    auto valid = [&](int64_t c) { return (int)min((int64_t)Q, a.L - c * Q); };

    // ---- forward sweep: the state entering every chunk; Sp = S after the last
    State G, Sp;
    zero(Sp);
    if (n > 0) {
        State st;
        if (seg > 0) load_map(st, a.Af + (slot - 1) * kMap, w);
        else if (a.init_state) load_np(st, a.init_state + bh * kMap, w);
        else zero(st);
        double x0, x1;
        sweep<R, true>(a, s, w, SW, cb, n - 1, st, Sst, &x0, &x1);
        if (last && a.dfinal) {   // (else the end state meets a zero gradient, or is the next segment's)
            sweep<R, true>(a, s, w, SW, cb + n - 1, 1, st, nullptr, &x0, &x1);
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int u = 0; u < 2; ++u) Sp[q][u] = st[q][u];
        }
    }
    if (!last) {
        load_map(Sp, a.Af + slot * kMap, w);
        load_map(G, a.Ar + (slot + 1) * kMap, w);
    } else if (a.dfinal) {
        load_np(G, a.dfinal + bh * kMap, w);
    } else {
        zero(G);
    }

    // ---- reverse
    const float Dh = a.D[s.h];
    double xdy = 0.0;   // (a chunk's terms in fp32, the segment's chunks in fp64: dD has no other rounding)
    float dAsum = 0.f;
    float pend_dt = 0.f, pend_lam = 0.f, first_dt = 0.f, first_lam = 0.f;   // (wave 0: chunk c + 1's first token)
    RawTok<R> raw;
    float ps[Shp<R>::TPS];
    float sc_dt = 0.f, sc_lam = 0.f, sc_A = 0.f;   // (wave 0: the current chunk's)
    Pair pB, pC;
    bf16x8 pX, pY;
    SBf sb;
    const int64_t ce = cb + n - 1, QH = Q * a.H;
    Cur u;
    u.t0 = ce * Q;
    u.th = s.tok + (u.t0 + w.wave * Shp<R>::TPS) * a.H;
    u.row = s.tok + (u.t0 + row_at<R>(w).t) * a.H;
    int64_t trow = s.tok + (u.t0 + (16 * w.it + w.l16) / R) * a.H;   // the output lane's token
    bf16 *dump = static_cast<bf16 *>(a.dump) + 8 * w.lane;   // (lanes past the end store here)
    // loads of chunk c, where the cursors stand; then to chunk c - 1 (kept at
    // the segment's first)
    auto fetch = [&](int64_t c) {
        const RowAt ra = row_at<R>(w);
        const int64_t at = u.row + past_end(ra.t, valid(c), Q, a.H);
        pB = load_pair<R>(ra, a.B, at);
        pC = load_pair<R>(ra, a.C, at);
        pX = load_row<R>(ra, a.x, at);
        pY = load_row<R>(ra, a.dy, at);
        u.row -= c == cb ? 0 : QH;
    };
    auto fetch_tok = [&](int64_t c) {
        load_tok<R>(a, s, w, u, valid(c), raw);
        u.th -= c == cb ? 0 : QH;
        u.t0 -= c == cb ? 0 : Q;
    };
    auto stage = [&](int nv, const h2 *cs, const Tok &o) {
        const RowAt ra = row_at<R>(w);
        float c[8], sn[8];
        cs_getn<8>(&cs[ra.t * LDC + ra.cp * 8], c, sn);
        if (nv < Q) {   // rows past the end are zero
            const bf16x8 z = {};
            if (ra.t >= nv) pB.lo = pB.hi = pC.lo = pC.hi = pX = pY = z;
        }
        put_rot(M.B, ra, pB, c, sn);
        put_rot(M.C, ra, pC, c, sn);
        put_tile_order(&M.X[ra.row * LDP], ra.cp, pX);
        put_tile_order(&M.Y[ra.row * LDP], ra.cp, pY);
        put_scaled(M.EY, ra, pY, o.ec[ra.row]);
    };
    if (n > 0) {
        const int nv = valid(ce);
        const int64_t c1 = max(ce - 1, cb);
        fetch_tok(ce);
        fetch(ce);
        sb = load_sbf(Sst + ce * kMap, w);
        __syncthreads();   // (the sweep's LDS)
        tok_scan<R>(a, w, ce, nv, raw, ps, M.seg, M.tok[0]);
        sc_dt = raw.dt; sc_lam = raw.lam; sc_A = raw.A;
        fetch_tok(c1);
        __syncthreads();
        tok_table<R>(w, nv, ps, M.seg, M.cs[0], M.tok[0]);
        __syncthreads();
        stage(nv, M.cs[0], M.tok[0]);
        fetch(c1);
        __syncthreads();
    }
    for (int64_t k = 0; k < n; ++k) {
        const int64_t c = ce - k, t0 = c * Q;
        const int nvalid = valid(c), par = (int)(k & 1);
        const int64_t c1 = max(c - 1, cb), c2 = max(c - 2, cb);   // (below the first: loaded unused)
        const int nv1 = valid(c1);
        const bool more = k + 1 < n;
        const Tok &o = M.tok[par];
        const h2 *cs = M.cs[par];
        // (the thread index is opaque from here, so that no address of the
        // chunk's work is held in registers across the loop)
        int tid = threadIdx.x;
        asm volatile("" : "+v"(tid));
        w = Lane(tid);
        const int J = w.it, hf = w.ph;
        const int row = 16 * J + w.l16, tl = row / R;   // this lane's chunk row and token

        // ======== region 0: state step, masked scores ========
        {
            const float e = exp2_fast(o.c2e), cn = o.ce[w.i], sn = o.se[w.i];
            float dps = 0.f, dcm = 0.f;
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                bf16x4 ur4, ui4, sr4, si4;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float gr = G[0][u][v], gi = G[1][u][v];
                    dps += gi * Sp[0][u][v] - gr * Sp[1][u][v];       // rotation of S_c by psi_e
                    const float ur = cn * gr + sn * gi, ui = cn * gi - sn * gr;
                    sr4[v] = sb.q[0][4 * u + v];
                    si4[v] = sb.q[1][4 * u + v];
                    const float sr = (float)sr4[v], si = (float)si4[v];
                    dcm += ur * sr + ui * si;                         // decay e^{cum_e} of S_{c-1}
                    ur4[v] = (bf16)ur;
                    ui4[v] = (bf16)ui;
                    G[0][u][v] = e * ur;
                    G[1][u][v] = e * ui;
                    Sp[0][u][v] = sr;
                    Sp[1][u][v] = si;
                }
                const int at = (16 * w.it + w.l16) * LDP + 16 * (2 * w.ph + u) + 4 * w.g;
                *reinterpret_cast<bf16x4 *>(&M.U[at]) = ur4;
                *reinterpret_cast<bf16x4 *>(&M.U[at + 64 * LDP]) = ui4;
                *reinterpret_cast<bf16x4 *>(&M.S[at]) = sr4;
                *reinterpret_cast<bf16x4 *>(&M.S[at + 64 * LDP]) = si4;
            }
            sb = load_sbf(Sst + c1 * kMap, w);
            dps = sum_g(dps);
            if (w.g == 0) M.dps[w.ph][w.i] = dps;
            dcm = sum_wave(e * dcm);
            if (w.lane == 0) M.dcm[w.wave] = dcm;
            add_outer(G, M.C, M.EY, w);
        }
        // fragments of the own rows (second operands below)
        bf16x8 fB[4], fX[2], fY[2];
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) fB[kk] = MM::load(&M.B[row * LDN + kk * 32 + 8 * w.g]);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            fX[kk] = MM::load(&M.X[row * LDP + kk * 32 + 8 * w.g]);
            fY[kk] = MM::load(&M.Y[row * LDP + kk * 32 + 8 * w.g]);
        }
        // column tiles (T, J), T >= J: lane element (t = 16 T + 4 g + v, j = row)
        bf16x8 wG[2], wD[2], wT[2];   // weighted scores as second operands, by pairs of tiles
        {
            const float c2j = o.c2[row], sgj = o.sig[row], gmj = o.gam[row];
            float colc = 0.f, cols = 0.f;
#pragma unroll
            for (int kp = 0; kp < 2; ++kp)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int T = 2 * kp + h;
                    f32x4 gt = {0.f, 0.f, 0.f, 0.f}, dg = gt;
                    if (T >= J) {
#pragma unroll
                        for (int kk = 0; kk < 4; ++kk)
                            gt = MM::mma(MM::load(&M.C[(16 * T + w.l16) * LDN + kk * 32 + 8 * w.g]), fB[kk], gt);
#pragma unroll
                        for (int kk = 0; kk < 2; ++kk)
                            dg = MM::mma(MM::load(&M.Y[(16 * T + w.l16) * LDP + kk * 32 + 8 * w.g]), fX[kk], dg);
                        const f32x4 c4 = *reinterpret_cast<const f32x4 *>(&o.c2[16 * T + 4 * w.g]);
                        float rv[TT];
#pragma unroll
                        for (int q = 0; q < TT; ++q) {
                            const int tt = (16 * T + 4 * w.g) / R + q;   // a token's rows
                            const bool off = tl < tt, on = tl == tt;
                            const float ex = off ? exp2_fast(c4[q * R] - c2j) : 0.f;
                            const float wt = off ? ex * sgj : on ? gmj : 0.f;
                            float dW = 0.f;   // dJ/dw summed over the token's rows
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                const int v = q * R + r;
                                dW += dg[v] * gt[v];
                                gt[v] *= wt;
                                dg[v] *= wt;
                            }
                            const float od = off ? dW : 0.f;
                            if (hf == 0) {   // (the halves share the sums)
                                rv[q] = od * wt;
                                colc += rv[q];
                            } else {
                                rv[q] = on ? dW : 0.f;
                                cols += od * ex;
                            }
                        }
                        if (hf == 0 || T == J) {
                            const float rs = sum16_each<TT>(rv, w.l16);
                            float *rd = hf == 0 ? M.rc[J] : M.rg;
                            if (w.l16 < TT) rd[16 * T + 4 * w.g + w.l16 * R] = rs;
                        }
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        wG[kp][4 * h + v] = (bf16)gt[v];
                        wD[kp][4 * h + v] = (bf16)dg[v];
                    }
                }
            if (hf == 0) {
                colc = sum_g(colc);
                if (w.g == 0) M.cc[row] = colc;
            } else {
                cols = sum_g(cols);
                if (w.g == 0) M.csg[row] = cols;
            }
        }
        // row tiles (Jt, J), Jt <= J, of dG^T: lane element (j = 16 Jt + 4 g + v, t = row)
        {
            const float c2t = o.c2[row], gmt = o.gam[row];
#pragma unroll
            for (int jp = 0; jp < 2; ++jp)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int Jt = 2 * jp + h;
                    f32x4 gT = {0.f, 0.f, 0.f, 0.f};
                    if (Jt <= J) {
#pragma unroll
                        for (int kk = 0; kk < 2; ++kk)
                            gT = MM::mma(MM::load(&M.X[(16 * Jt + w.l16) * LDP + kk * 32 + 8 * w.g]), fY[kk], gT);
                        const f32x4 c4 = *reinterpret_cast<const f32x4 *>(&o.c2[16 * Jt + 4 * w.g]);
                        const f32x4 s4 = *reinterpret_cast<const f32x4 *>(&o.sig[16 * Jt + 4 * w.g]);
#pragma unroll
                        for (int q = 0; q < TT; ++q) {
                            const int tj = (16 * Jt + 4 * w.g) / R + q;
                            float wt = tj < tl ? exp2_fast(c2t - c4[q * R]) * s4[q * R] : 0.f;
                            wt = tj == tl ? gmt : wt;
#pragma unroll
                            for (int r = 0; r < R; ++r) gT[q * R + r] *= wt;
                        }
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) wT[jp][4 * h + v] = (bf16)gT[v];
                }
        }
        tok_scan<R>(a, w, c1, nv1, raw, ps, M.seg, M.tok[par ^ 1]);
        const float nx_dt = raw.dt, nx_lam = raw.lam, nx_A = raw.A;
        fetch_tok(c2);
        __syncthreads();

        // ======== region 1: the chunk's gradients ========
        const float vj = o.v[row], ec = o.ec[row];
        const int rk = row % R;
        // (every lane stores, so that a wait for the loads before never waits for these stores)
        bf16 *gx = static_cast<bf16 *>(a.dx) + (trow * R + rk) * kP + 32 * hf + 8 * w.g;
        bf16 *gB = static_cast<bf16 *>(a.dB) + (trow * R + rk) * kN + 32 * hf + 8 * w.g;
        bf16 *gC = static_cast<bf16 *>(a.dC) + (trow * R + rk) * kN + 32 * hf + 8 * w.g;
        if (nvalid < Q) {
            asm volatile("");
            if (tl >= nvalid) gx = gB = gC = dump;
        }
        {
            // dx: columns 32 hf + 8 g + e
            f32x4 d[2], bu[2];
#pragma unroll
            for (int ab = 0; ab < 2; ++ab) {
                d[ab] = bu[ab] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kp = 0; kp < 2; ++kp)
                    if (2 * kp + 1 >= J) d[ab] = MM::mma(load_kt2(M.Y, LDP, 32 * kp, 32 * hf + 16 * ab, w.g, w.l16), wG[kp], d[ab]);
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    bu[ab] = MM::mma(load_kt(M.U, LDP, 32 * kk, 32 * hf + 16 * ab, w.g, w.l16), fB[kk], bu[ab]);
            }
            const bf16x8 xv = get_tile_order(&M.X[row * LDP], 4 * hf + w.g);
            const bf16x8 yv = get_tile_order(&M.Y[row * LDP], 4 * hf + w.g);
            float dvp = 0.f, xy = 0.f;
            bf16x8 out;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float xe = (float)xv[e], ye = (float)yv[e], be = bu[e / 4][e % 4];
                dvp += xe * be;
                xy += xe * ye;
                out[e] = (bf16)(d[e / 4][e % 4] + vj * be + Dh * ye);
            }
            *reinterpret_cast<bf16x8 *>(gx) = out;
            xdy += (double)xy;
            dvp = sum_g(dvp);
            if (w.g == 0) M.dv[hf][row] = dvp;
        }
        float cn[8], sn[8], dpsi[8];
        cs_getn<8>(&cs[tl * LDC + 32 * hf + 8 * w.g], cn, sn);
        {
            // dB: pairs i = 32 hf + 8 g + e
            f32x4 d[2][2], xu[2][2];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int ab = 0; ab < 2; ++ab) {
                    d[q][ab] = xu[q][ab] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kp = 0; kp < 2; ++kp)
                        if (2 * kp + 1 >= J)
                            d[q][ab] = MM::mma(load_kt2(M.C, LDN, 32 * kp, 64 * q + 32 * hf + 16 * ab, w.g, w.l16), wD[kp], d[q][ab]);
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
                        xu[q][ab] = MM::mma(MM::load(&M.U[(64 * q + 32 * hf + 16 * ab + w.l16) * LDP + 32 * kk + 8 * w.g]), fX[kk], xu[q][ab]);
                }
            const bf16x8 br = get_tile_order(&M.B[row * LDN], 4 * hf + w.g);
            const bf16x8 bi = get_tile_order(&M.B[row * LDN + kNH], 4 * hf + w.g);
            bf16x8 o0, o1;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float re = d[0][e / 4][e % 4] + vj * xu[0][e / 4][e % 4];
                const float im = d[1][e / 4][e % 4] + vj * xu[1][e / 4][e % 4];
                dpsi[e] = re * (float)bi[e] - im * (float)br[e];
                o0[e] = (bf16)(cn[e] * re - sn[e] * im);
                o1[e] = (bf16)(sn[e] * re + cn[e] * im);
            }
            *reinterpret_cast<bf16x8 *>(gB) = o0;
            *reinterpret_cast<bf16x8 *>(gB + kNH) = o1;
        }
        {
            // dC
            f32x4 d[2][2], t2[2][2];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int ab = 0; ab < 2; ++ab) {
                    d[q][ab] = t2[q][ab] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int jp = 0; jp < 2; ++jp)
                        if (2 * jp <= J)
                            d[q][ab] = MM::mma(load_kt2(M.B, LDN, 32 * jp, 64 * q + 32 * hf + 16 * ab, w.g, w.l16), wT[jp], d[q][ab]);
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
                        t2[q][ab] = MM::mma(MM::load(&M.S[(64 * q + 32 * hf + 16 * ab + w.l16) * LDP + 32 * kk + 8 * w.g]), fY[kk], t2[q][ab]);
                }
            const bf16x8 cr = get_tile_order(&M.C[row * LDN], 4 * hf + w.g);
            const bf16x8 ci = get_tile_order(&M.C[row * LDN + kNH], 4 * hf + w.g);
            float dcy = 0.f;
            bf16x8 o0, o1;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float tr = t2[0][e / 4][e % 4], ti = t2[1][e / 4][e % 4];
                const float re = d[0][e / 4][e % 4] + ec * tr, im = d[1][e / 4][e % 4] + ec * ti;
                dcy += (float)cr[e] * tr + (float)ci[e] * ti;
                dpsi[e] += re * (float)ci[e] - im * (float)cr[e];
                o0[e] = (bf16)(cn[e] * re - sn[e] * im);
                o1[e] = (bf16)(sn[e] * re + cn[e] * im);
            }
            *reinterpret_cast<bf16x8 *>(gC) = o0;
            *reinterpret_cast<bf16x8 *>(gC + kNH) = o1;
            dcy = sum_g(dcy);
            if (w.g == 0) M.dcy[hf][row] = ec * dcy;
        }
        // angle gradients: suffix sums over the tile's tokens, tile totals to LDS
#pragma unroll
        for (int e = 0; e < 8; ++e) dpsi[e] = suffix16<R>(sum_rank<R>(dpsi[e]));
        if (w.l16 == 0) {
#pragma unroll
            for (int e = 0; e < 8; e += 4)
                *reinterpret_cast<f32x4 *>(&M.dth[J][32 * hf + 8 * w.g + e]) =
                    f32x4{dpsi[e], dpsi[e + 1], dpsi[e + 2], dpsi[e + 3]};
        }
        tok_table<R>(w, nv1, ps, M.seg, M.cs[par ^ 1], M.tok[par ^ 1]);
        __syncthreads();

        // ======== region 2: next rows, dtheta, per-token scalars ========
        stage(nv1, M.cs[par ^ 1], M.tok[par ^ 1]);
        fetch(c2);
        if (w.l16 % R == 0 && tl < nvalid) {
            // (dps: the state's rotation by psi_e, which every token's angle enters)
#pragma unroll
            for (int e = 0; e < 8; e += 4) {
                const int i = 32 * hf + 8 * w.g + e;
                f32x4 off = *reinterpret_cast<const f32x4 *>(&M.dps[0][i]) +
                            *reinterpret_cast<const f32x4 *>(&M.dps[1][i]);
                for (int q = J + 1; q < 4; ++q) off += *reinterpret_cast<const f32x4 *>(&M.dth[q][i]);
                f32x4u out;
#pragma unroll
                for (int v = 0; v < 4; ++v) out[v] = dpsi[e + v] + off[v];
                *reinterpret_cast<f32x4u *>(a.dtheta + trow * kNH + i) = out;
            }
        }
        if (w.wave == 0) {
            const int rw = w.lane, t = rw / R;   // lane: a row; a token's R lanes agree after the sums
            const bool lead = rw % R == 0, in = t < nvalid;
            const float dvr = M.dv[0][rw] + M.dv[1][rw], vt = o.v[rw];
            const float et = in ? exp2_fast(o.c2e - o.c2[rw]) : 0.f;   // v_t / sigma_t
            float dcum = M.dcy[0][rw] + M.dcy[1][rw] - M.cc[rw] - dvr * vt;
            float dsig = M.csg[rw] + dvr * et;
            dcum = sum_rank<R>(dcum);
            dsig = sum_rank<R>(dsig);
            for (int q = 0; q <= rw / 16; ++q) dcum += M.rc[q][t * R];
            // dcum_e: the v_j terms and the state's decay
            float cend = sum_wave(dvr * vt + (rw < kNW ? M.dcm[rw] : 0.f));
            if (t == nvalid - 1) dcum += cend;
            // d(dt_u A_u) = sum_{t >= u} dcum_t: a scan in reverse lane order
            const float rv = __shfl(lead && in ? dcum : 0.f, kWave - 1 - rw, kWave);
            const float da = __shfl(lane_scan(rv), kWave - 1 - rw, kWave);
            const float dsig_prev = __shfl(dsig, max(rw - R, 0), kWave);
            const float dgam = M.rg[t * R] + dsig;   // sigma_t = gamma_t + ...
            float ddt = sc_A * da + sc_lam * dgam, dl = sc_dt * dgam;
            if (t > 0) {   // the previous token's sigma reads this token's lambda and dt
                ddt += (1.f - sc_lam) * dsig_prev;
                dl -= sc_dt * dsig_prev;
            }
            const int64_t at = s.tok + (t0 + t) * a.H;
            if (lead && in) {
                if (t > 0) {   // (token 0 waits for the chunk before it)
                    a.ddt[at] = ddt;
                    a.dlam[at] = dl;
                }
                const float dAt = sc_dt * da;
                dAsum += dAt;
                if (a.dA_per_token) a.dA[at] = dAt;
            }
            // the sigma of this chunk's last token reaches the first token of
            // the chunk worked on before
            const float dse = lane_bcast(dsig, nvalid * R - 1);
            if (w.lane == 0) {
                if (k > 0) {
                    a.ddt[at + Q * a.H] = pend_dt + (1.f - first_lam) * dse;
                    a.dlam[at + Q * a.H] = pend_lam - first_dt * dse;
                } else {
                    a.dsig[slot] = dse;
                }
                if (!more) {   // (k_bwd_finish adds the segment before's)
                    a.ddt[at] = ddt;
                    a.dlam[at] = dl;
                }
            }
            pend_dt = ddt;
            pend_lam = dl;
            first_dt = sc_dt;
            first_lam = sc_lam;
            sc_dt = nx_dt;
            sc_lam = nx_lam;
            sc_A = nx_A;
        }
        trow -= QH;
        __syncthreads();
    }
    if (seg == 0 && a.dinit) store_np(G, a.dinit + bh * kMap, w);
    // per-segment partials of dD and dA
    const float xs = sum_wave((float)xdy);
    if (w.lane == 0) M.red[w.wave] = xs;
    dAsum = sum_wave(dAsum);
    __syncthreads();
    if (w.tid == 0) {
        float d = 0.f;
        for (int q = 0; q < kNW; ++q) d += M.red[q];
        a.dDpart[slot] = d;
        a.dApart[slot] = dAsum;
    }
}

// ---------------------------------------------------------------------------
// k_bwd_finish: blocks 0 .. H - 1 the per-head sums of the segments' partials
// in a fixed order; the rest the sigma term of each segment's last token in
// the next segment's first token (sigma_e = gamma_e + (1 - lambda_{e+1}) dt_{e+1}).
// ---------------------------------------------------------------------------
constexpr int kThrF = 256;
__global__ __launch_bounds__(kThrF) void k_bwd_finish(BwdArgs a, int Q) {
    __shared__ double s_a[kThrF], s_d[kThrF];
    const int tid = threadIdx.x;
    if (blockIdx.x >= a.H) {
        const int64_t q = ((int64_t)blockIdx.x - a.H) * kThrF + tid;
        if (q >= a.batch * a.H * (a.nseg - 1)) return;
        const int64_t bh = q / (a.nseg - 1), seg = q % (a.nseg - 1) + 1;
        const int64_t k = slice_of(a, bh).tok + seg * a.G * Q * a.H;
        const float d = a.dsig[bh * a.nseg + seg - 1];
        a.ddt[k] += (1.f - a.lam[k]) * d;
        a.dlam[k] -= a.dt[k] * d;
        return;
    }
    const int64_t h = blockIdx.x, n = a.batch * a.nseg;
    double sa = 0.0, sd = 0.0;
    for (int64_t q = tid; q < n; q += kThrF) {
        const int64_t s = (q / a.nseg * a.H + h) * a.nseg + q % a.nseg;
        sa += a.dApart[s];
        sd += a.dDpart[s];
    }
    s_a[tid] = sa;
    s_d[tid] = sd;
    __syncthreads();
    for (int w = kThrF / 2; w > 0; w >>= 1) {
        if (tid < w) {
            s_a[tid] += s_a[tid + w];
            s_d[tid] += s_d[tid + w];
        }
        __syncthreads();
    }
    if (tid == 0) {
        a.dD[h] = (float)s_d[0];
        if (!a.dA_per_token) a.dA[h] = (float)s_a[0];
    }
}

// Store target of the lanes past the end: 16 bytes a lane, twice kNH apart.
constexpr size_t kDumpBytes = 2 * kNH + 16 * kWave;

// Most segments a slice may be split into: the workspace holds their maps, so
// the bound does not depend on the device.
constexpr int64_t kMaxGroups = 1024;
int64_t max_segments(int64_t BH, int64_t nchunks) {
    return std::max<int64_t>(1, std::min(nchunks, kMaxGroups / BH));
}

// Chunks per segment: the least estimated time over the segment counts.  A
// workgroup of k_bwd_main takes a CU and about kMain a chunk; several
// segments a slice add two aggregate sweeps (kAggr a chunk, two workgroups a
// CU) and the fold over the segments.
int64_t choose_chunks(int64_t BH, int64_t nchunks, int ncu) {
    constexpr double kMain = 10.0, kAggr = 3.0, kPass = 8.0, kFold = 0.25;   // us
    const int64_t most = max_segments(BH, nchunks);
    double best = 0.0;
    int64_t bestG = nchunks;
    for_segment_counts(most, BH, ncu, [&](int64_t ns) {
        const int64_t G = (nchunks + ns - 1) / ns, m = (nchunks + G - 1) / G;
        double t = (double)((BH * m + ncu - 1) / ncu) * G * kMain;
        if (m > 1) t += (double)((BH * (m - 1) * 2 + 2 * ncu - 1) / (2 * ncu)) * G * kAggr + kPass + kFold * m;
        if (ns == 1 || t < best) {
            best = t;
            bestG = G;
        }
    });
    return bestG;
}

template <int R>
hipError_t launch_bwd(const BwdArgs &args, hipStream_t stream) {
    constexpr int Q = Shp<R>::Q;
    static int cus[64];
    BwdArgs a = args;
    const int64_t BH = a.batch * a.H;
    a.G = 1;
    a.nseg = 1;
    if (a.nchunks > 0) {
        const int ncu = cu_count(cus);
        if (ncu <= 0) return hipErrorInvalidDevice;
        a.G = choose_chunks(BH, a.nchunks, ncu);
        a.nseg = (a.nchunks + a.G - 1) / a.G;
    }
    const unsigned ns = (unsigned)a.nseg, nsl = (unsigned)BH;
    if (a.nseg > 1) {
        hipLaunchKernelGGL((k_bwd_aggr<R>), dim3(nsl, ns - 1, 2), dim3(kThr), 0, stream, a);
        hipLaunchKernelGGL(k_bwd_pass, dim3(nsl, 2, 2), dim3(kThr), 0, stream, a);
    }
    hipLaunchKernelGGL((k_bwd_main<R>), dim3(nsl, ns), dim3(kThr), 0, stream, a);
    const int64_t edges = (BH * (a.nseg - 1) + kThrF - 1) / kThrF;
    hipLaunchKernelGGL(k_bwd_finish, dim3((unsigned)(a.H + edges)), dim3(kThrF), 0, stream, a, Q);
    return hipGetLastError();
}

}  // namespace

BwdWorkspaceLayout bwd_workspace_layout(int64_t BH, int64_t nchunks, int64_t N, int64_t P) {
    auto up = [](size_t v) { return (v + 255) / 256 * 256; };
    const size_t np = (size_t)(N * P), segs = (size_t)BH * (size_t)max_segments(BH, nchunks);
    BwdWorkspaceLayout w = {};
    w.off_Af = kCtlBytes;   // (the scans' control block, left untouched in a shared workspace)
    w.off_Ar = up(w.off_Af + segs * np * sizeof(float));
    w.off_Sst = up(w.off_Ar + segs * np * sizeof(float));
    w.off_tot = up(w.off_Sst + (size_t)BH * (size_t)nchunks * np * 2);
    w.off_dump = up(w.off_tot + segs * 2 * kTot * sizeof(float));
    w.off_dsig = up(w.off_dump + kDumpBytes);
    w.off_dA = up(w.off_dsig + segs * sizeof(float));
    w.off_dD = up(w.off_dA + segs * sizeof(float));
    // (at least the documented three fp32 maps a chunk)
    w.total = up(std::max(w.off_dD + segs * sizeof(float),
                          kCtlBytes + (size_t)BH * (size_t)nchunks * 3 * np * sizeof(float)));
    return w;
}

bwd_launch_fn find_bwd_impl(int io, int64_t N, int64_t P, int64_t R, int64_t Q) {
    if (io != 1 || N != kN || P != kP || R * Q != kRows) return nullptr;
    if (R == 1) return &launch_bwd<1>;
    if (R == 2) return &launch_bwd<2>;
    if (R == 4) return &launch_bwd<4>;
    return nullptr;
}

}  // namespace m3

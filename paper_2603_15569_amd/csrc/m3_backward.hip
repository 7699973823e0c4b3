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
// carrying the state through a segment in registers takes 2.90 ms and 175 us.
// Operands are bf16 with fp32 accumulation (as the forward); the carried
// state and gradient, the prefix sums, weights and every scalar gradient are
// fp32.  Results are deterministic: no atomics.
#include <algorithm>

#include "m3_device.h"
#include "m3_internal.h"
#include "m3_scan_common.h"

namespace m3 {
namespace {

using namespace scan;

constexpr int kN = 128, kP = 64, kNH = 64, kRows = 64;
constexpr int kNW = 8, kThr = kNW * kWave;
constexpr int LDN = kN + 8;   // bf16 row strides (16-byte padding)
constexpr int LDP = kP + 8;
constexpr int kMap = kN * kP;
constexpr float kLog2e = 1.44269504088896340736f;
typedef Mma<bf16> MM;
// four floats at 4-byte alignment (the angles' arrays need no more)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Lane and wave coordinates of a 512-thread workgroup.  The carried N x P
// state is held transposed in MFMA tiles: wave (it, ph) owns the pair tiles
// n = 16 it + l16 (q = 0) and 64 + 16 it + l16 (q = 1) and the columns
// p = 16 (2 ph + u) + 4 g + v, element st[q][u][v].
struct Lane {
    int tid, lane, wave, g, l16, it, ph;
    __device__ __forceinline__ Lane() : Lane((int)threadIdx.x) {}
    __device__ __forceinline__ explicit Lane(int tid_) {
        tid = tid_;
        lane = tid & (kWave - 1);
        wave = __builtin_amdgcn_readfirstlane(tid / kWave);
        g = lane >> 4;
        l16 = lane & 15;
        it = wave & 3;
        ph = wave >> 2;
    }
};
typedef f32x4 State[2][2];

// A chunk's scalars by row (token, rank): base-2 log-decay prefix, gamma,
// sigma, v, e^{cum}; its total log-decay and the pairs' total angles.
struct Tok {
    float c2[kRows], gam[kRows], sig[kRows], v[kRows], ec[kRows];
    float psie[kNH];
    float c2e;
};

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

// Raw values of a chunk's prologue: wave w's tokens w TPS .. of the angles
// (pair = lane), and, by wave 0 with one lane a row, the token's scalars.
template <int R> struct RawTok {
    float th[Shp<R>::TPS];
    float dt, lam, A, dtn, lamn;
};

template <int R>
__device__ __forceinline__ void load_tok(const BwdArgs &a, const Slice &s, const Lane &w, int64_t c, int nvalid,
                                         RawTok<R> &r) {
    constexpr int Q = Shp<R>::Q, TPS = Shp<R>::TPS;
    const int64_t t0 = c * Q;
    const float *th = a.theta + (s.tok + t0 * a.H) * kNH + w.lane;
#pragma unroll
    for (int k = 0; k < TPS; ++k) {
        const int t = min(w.wave * TPS + k, nvalid - 1);
        r.th[k] = th[(int64_t)t * a.H * kNH];
    }
    if (w.wave == 0) {
        const int t = min(w.lane / R, nvalid - 1);
        const int64_t tg = t0 + t, tn = min(tg + 1, a.L - 1);
        r.dt = a.dt[s.tok + tg * a.H];
        r.lam = a.lam[s.tok + tg * a.H];
        r.A = a.A[s.b * a.a_sb + tg * a.a_st + s.h * a.a_sh];
        r.dtn = a.dt[s.tok + tn * a.H];
        r.lamn = a.lam[s.tok + tn * a.H];
    }
}

// Step 1: each wave's angle prefix sums (in place, its total to `seg`), and
// wave 0 the scalar tables.  Tokens past the end of the sequence get zero
// angles and weights.
template <int R>
__device__ __forceinline__ void tok_scan(const BwdArgs &a, const Lane &w, int64_t c, int nvalid, RawTok<R> &r,
                                         float (*seg)[kNH], Tok &o) {
    constexpr int Q = Shp<R>::Q, TPS = Shp<R>::TPS;
    float run = 0.f;
#pragma unroll
    for (int k = 0; k < TPS; ++k) {
        run += w.wave * TPS + k < nvalid ? r.th[k] : 0.f;
        r.th[k] = run;
    }
    seg[w.wave][w.lane] = run;
    if (w.wave == 0) {
        const int t = w.lane / R;
        const bool in = t < nvalid;
        const float cum = lane_scan(in && w.lane % R == 0 ? r.dt * r.A : 0.f);
        const float c2 = cum * kLog2e, c2e = lane_bcast(c2, nvalid * R - 1);
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

// Step 2: the cos / sin table of psi_t and psi_e.
template <int R>
__device__ __forceinline__ void tok_table(const Lane &w, int nvalid, const RawTok<R> &r, const float (*seg)[kNH],
                                          h2 *cs, Tok &o) {
    constexpr int TPS = Shp<R>::TPS;
    float off = 0.f;
    for (int s = 0; s < w.wave; ++s) off += seg[s][w.lane];
#pragma unroll
    for (int k = 0; k < TPS; ++k) {
        const int t = w.wave * TPS + k;
        const float psi = r.th[k] + off;
        float sn, cn;
        sincos_fast(psi, &sn, &cn);
        cs_put(&cs[t * kNH + w.lane], cn, sn);
        if (t == nvalid - 1) o.psie[w.lane] = psi;
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
// B or C piece pair (channels i and i + N/2) of the thread's row.
struct Pair { bf16x8 lo, hi; };
template <int R>
__device__ __forceinline__ Pair load_pair(const BwdArgs &a, const Slice &s, const RowAt &k, const void *src,
                                          int64_t t0, int nvalid) {
    const int64_t t = t0 + min(k.t, nvalid - 1);
    const bf16 *p = static_cast<const bf16 *>(src) + ((s.tok + t * a.H) * R + k.r) * kN + k.cp * 8;
    return Pair{*reinterpret_cast<const bf16x8 *>(p), *reinterpret_cast<const bf16x8 *>(p + kNH)};
}
template <int R>
__device__ __forceinline__ bf16x8 load_row(const BwdArgs &a, const Slice &s, const RowAt &k, const void *src,
                                           int64_t t0, int nvalid) {
    const int64_t t = t0 + min(k.t, nvalid - 1);
    return *reinterpret_cast<const bf16x8 *>(static_cast<const bf16 *>(src) +
                                             ((s.tok + t * a.H) * R + k.r) * kP + k.cp * 8);
}
// Rotated by -psi_t (cos c, sin s of the thread's eight pairs) into [row][LDN].
__device__ __forceinline__ void put_rot(bf16 *dst, const RowAt &k, Pair v, const float (&c)[8], const float (&s)[8],
                                        bool in) {
    Pair o;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const float u = in ? (float)v.lo[e] : 0.f, x = in ? (float)v.hi[e] : 0.f;
        o.lo[e] = (bf16)(c[e] * u + s[e] * x);
        o.hi[e] = (bf16)(c[e] * x - s[e] * u);
    }
    *reinterpret_cast<bf16x8 *>(&dst[k.row * LDN + k.cp * 8]) = o.lo;
    *reinterpret_cast<bf16x8 *>(&dst[k.row * LDN + kNH + k.cp * 8]) = o.hi;
}
__device__ __forceinline__ void put_row(bf16 *dst, const RowAt &k, bf16x8 v, bool in) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = in ? v[e] : (bf16)0.f;
    *reinterpret_cast<bf16x8 *>(&dst[k.row * LDP + k.cp * 8]) = v;
}
__device__ __forceinline__ void put_row_scaled(bf16 *dst, const RowAt &k, bf16x8 v, float sc, bool in) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = in ? (bf16)(sc * (float)v[e]) : (bf16)0.f;
    *reinterpret_cast<bf16x8 *>(&dst[k.row * LDP + k.cp * 8]) = v;
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
                &m[(64 * q + 16 * w.it + w.l16) * kP + 16 * (2 * w.ph + u) + 4 * w.g]);
}
__device__ __forceinline__ void store_np(const State &st, float *m, const Lane &w) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int u = 0; u < 2; ++u)
            *reinterpret_cast<f32x4 *>(
                &m[(64 * q + 16 * w.it + w.l16) * kP + 16 * (2 * w.ph + u) + 4 * w.g]) = st[q][u];
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
// Returns the sums of cum_e (base 2) and of the lane's psi_e.  Two barriers a
// chunk; the next chunk's rows and the angles of the one after are in flight
// while a chunk is worked on.
// ---------------------------------------------------------------------------
template <int R> struct SweepLds {
    bf16 rows[kRows * LDN], cols[kRows * LDP];
    h2 cs[Shp<R>::Q * kNH];
    float seg[kNW][kNH];
    Tok tok[4];
};

template <int R, bool kFwd>
__device__ __forceinline__ void sweep(const BwdArgs &a, const Slice &s, const Lane &w, SweepLds<R> &L, int64_t c0,
                                      int64_t n, State &st, bf16 *Sst, float *sum_c2, float *sum_psi) {
    constexpr int Q = Shp<R>::Q;
    const void *rsrc = kFwd ? a.B : a.C, *csrc = kFwd ? a.x : a.dy;
    const RowAt ra = row_at<R>(w);
    auto chunk = [&](int64_t k) { return kFwd ? c0 + k : c0 - k; };
    auto valid = [&](int64_t c) { return (int)min((int64_t)Q, a.L - c * Q); };
    RawTok<R> raw;
    Pair pr;
    bf16x8 px;
    *sum_c2 = 0.f;
    *sum_psi = 0.f;
    if (n > 0) {
        load_tok<R>(a, s, w, chunk(0), valid(chunk(0)), raw);
        pr = load_pair<R>(a, s, ra, rsrc, chunk(0) * Q, valid(chunk(0)));
        px = load_row<R>(a, s, ra, csrc, chunk(0) * Q, valid(chunk(0)));
        tok_scan<R>(a, w, chunk(0), valid(chunk(0)), raw, L.seg, L.tok[0]);
        __syncthreads();
    }
    for (int64_t k = -1; k < n; ++k) {
        // (a) chunk k's state update; the table of chunk k + 1
        if (k >= 0) {
            const Tok &o = L.tok[k & 3];
            if (Sst) store_sbf(Sst + chunk(k) * kMap, to_bf(st), w);
            const float psi = o.psie[16 * w.it + w.l16], e = exp2_fast(o.c2e);
            float sn, cn;
            sincos_fast(psi, &sn, &cn);
            *sum_c2 += o.c2e;
            *sum_psi += psi;
            if constexpr (!kFwd) rotate(st, cn, -sn);
            scale(st, e);
            add_outer(st, L.rows, L.cols, w);
            if constexpr (kFwd) rotate(st, cn, sn);
        }
        const int64_t c1 = chunk(k + 1);
        const bool more = k + 1 < n;
        const int nv1 = more ? valid(c1) : 0;
        if (more) {
            tok_table<R>(w, nv1, raw, L.seg, L.cs, L.tok[(k + 1) & 3]);
            if (k + 2 < n) load_tok<R>(a, s, w, chunk(k + 2), valid(chunk(k + 2)), raw);
        }
        __syncthreads();
        // (b) chunk k + 1's rows staged; the scans of chunk k + 2
        if (more) {
            const Tok &o = L.tok[(k + 1) & 3];
            float c[8], sn[8];
            cs_getn<8>(&L.cs[ra.t * kNH + ra.cp * 8], c, sn);
            put_rot(L.rows, ra, pr, c, sn, ra.t < nv1);
            put_row_scaled(L.cols, ra, px, kFwd ? o.v[ra.row] : o.ec[ra.row], ra.t < nv1);
            if (k + 2 < n) {
                const int64_t c2 = chunk(k + 2);
                const int nv2 = valid(c2);
                pr = load_pair<R>(a, s, ra, rsrc, c2 * Q, nv2);
                px = load_row<R>(a, s, ra, csrc, c2 * Q, nv2);
                tok_scan<R>(a, w, c2, nv2, raw, L.seg, L.tok[(k + 2) & 3]);
            }
        }
        __syncthreads();
    }
    if (Sst) store_sbf(Sst + chunk(n) * kMap, to_bf(st), w);
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
    float sc, sp;
    if (fwd) sweep<R, true>(a, s, w, L, c0, n, st, nullptr, &sc, &sp);
    else sweep<R, false>(a, s, w, L, c0 + n - 1, n, st, nullptr, &sc, &sp);
    const int64_t slot = bh * a.nseg + seg;
    store_map(st, (fwd ? a.Af : a.Ar) + slot * kMap, w);
    float *tot = a.tot + (slot * 2 + (fwd ? 0 : 1)) * (1 + kNH);
    if (w.ph == 0 && w.g == 0) tot[1 + 16 * w.it + w.l16] = sp;
    if (w.tid == 0) tot[0] = sc;
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
        const float *m = src + bh * kMap + 16 * (2 * w.ph + u) + 4 * w.g;
        re = *reinterpret_cast<const f32x4 *>(&m[(16 * w.it + w.l16) * kP]);
        im = *reinterpret_cast<const f32x4 *>(&m[(64 + 16 * w.it + w.l16) * kP]);
    }
    float *M = fwd ? a.Af : a.Ar;
    const int n = (int)a.nseg - 1;
    constexpr int DEPTH = 4;   // segments whose loads are issued together
    for (int k0 = 0; k0 < n; k0 += DEPTH) {
        f32x4 mr[DEPTH], mi[DEPTH];
        float c2[DEPTH], ps[DEPTH];
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int k = min(k0 + d, n - 1);
            const int64_t slot = bh * a.nseg + (fwd ? k : a.nseg - 1 - k);
            const float *tot = a.tot + (slot * 2 + (fwd ? 0 : 1)) * (1 + kNH);
            c2[d] = tot[0];
            ps[d] = tot[1 + 16 * w.it + w.l16];
            const float *m = M + slot * kMap + 4 * w.tid;
            mr[d] = *reinterpret_cast<const f32x4 *>(&m[u * 4 * kThr]);
            mi[d] = *reinterpret_cast<const f32x4 *>(&m[(2 + u) * 4 * kThr]);
        }
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            if (k0 + d >= n) break;
            const int64_t slot = bh * a.nseg + (fwd ? k0 + d : a.nseg - 1 - (k0 + d));
            const float e = exp2_fast(c2[d]);
            float sn, cn;
            sincos_fast(ps[d], &sn, &cn);
            if (!fwd) sn = -sn;
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
// transposed, from operands whose rows are permuted (perm_*), so a lane holds
// eight consecutive channels of one row: 16-byte stores, the row's weights
// are per-lane scalars, and the sums over a row are in-lane.
// ---------------------------------------------------------------------------
template <int R> struct MainLds {
    bf16 B[kRows * LDN], C[kRows * LDN];
    bf16 X[kRows * LDP], Y[kRows * LDP], EY[kRows * LDP];   // x, dy, e^{cum} dy
    bf16 S[kN * LDP], U[kN * LDP];                          // S_{c-1}, U_c  [n][p]
    h2 cs[2][Shp<R>::Q * kNH];
    Tok tok[2];
    float seg[kNW][kNH];
    float rc[4][kRows], rg[kRows];     // sums of the mask terms by token row group
    float cc[kRows], csg[kRows];       // by column: cum, sigma
    float dv[2][kRows], dcy[2][kRows]; // dJ/dv_j and the y state term of cum_t, by half
    float dps[2][kNH], dcm[kNW];       // state terms of psi_e (by column half) and cum_e
    float dth[4][kNH];                 // dpsi totals of the row tiles
    float red[kNW];
};

template <int R>
__global__ __launch_bounds__(kThr, 2) void k_bwd_main(BwdArgs a) {
    constexpr int Q = Shp<R>::Q;
    constexpr int TT = 4 / R;   // tokens among a lane's four accumulator rows
    __shared__ __attribute__((aligned(16))) char mem[std::max(sizeof(SweepLds<R>), sizeof(MainLds<R>))];
    SweepLds<R> &SW = *reinterpret_cast<SweepLds<R> *>(mem);
    MainLds<R> &M = *reinterpret_cast<MainLds<R> *>(mem);
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
        float x0, x1;
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
    float xdy = 0.f, dAsum = 0.f;
    float pend_dt = 0.f, pend_lam = 0.f, first_dt = 0.f, first_lam = 0.f;   // (wave 0: chunk c + 1's first token)
    RawTok<R> raw;
    float sc_dt = 0.f, sc_lam = 0.f, sc_A = 0.f;   // (wave 0: the current chunk's)
    Pair pB, pC;
    bf16x8 pX, pY;
    SBf sb;
    auto load_rows = [&](int64_t c) {
        const RowAt ra = row_at<R>(w);
        const int nv = valid(c);
        pB = load_pair<R>(a, s, ra, a.B, c * Q, nv);
        pC = load_pair<R>(a, s, ra, a.C, c * Q, nv);
        pX = load_row<R>(a, s, ra, a.x, c * Q, nv);
        pY = load_row<R>(a, s, ra, a.dy, c * Q, nv);
    };
    auto stage = [&](int nv, const h2 *cs, const Tok &o) {
        const RowAt ra = row_at<R>(w);
        const bool in = ra.t < nv;
        float c[8], sn[8];
        cs_getn<8>(&cs[ra.t * kNH + ra.cp * 8], c, sn);
        put_rot(M.B, ra, pB, c, sn, in);
        put_rot(M.C, ra, pC, c, sn, in);
        put_row(M.X, ra, pX, in);
        put_row(M.Y, ra, pY, in);
        put_row_scaled(M.EY, ra, pY, o.ec[ra.row], in);
    };
    const int64_t ce = cb + n - 1;
    if (n > 0) {
        const int nv = valid(ce);
        load_tok<R>(a, s, w, ce, nv, raw);
        load_rows(ce);
        sb = load_sbf(Sst + ce * kMap, w);
        __syncthreads();   // (the sweep's LDS)
        tok_scan<R>(a, w, ce, nv, raw, M.seg, M.tok[0]);
        __syncthreads();
        tok_table<R>(w, nv, raw, M.seg, M.cs[0], M.tok[0]);
        sc_dt = raw.dt; sc_lam = raw.lam; sc_A = raw.A;
        if (n > 1) load_tok<R>(a, s, w, ce - 1, valid(ce - 1), raw);
        __syncthreads();
        stage(nv, M.cs[0], M.tok[0]);
        if (n > 1) load_rows(ce - 1);
        __syncthreads();
    }
    for (int64_t k = 0; k < n; ++k) {
        const int64_t c = ce - k, t0 = c * Q;
        const int nvalid = valid(c), par = (int)(k & 1);
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
            const float psi = o.psie[16 * w.it + w.l16], e = exp2_fast(o.c2e);
            float sn, cn;
            sincos_fast(psi, &sn, &cn);
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
            if (more) sb = load_sbf(Sst + (c - 1) * kMap, w);
            dps = sum_g(dps);
            if (w.g == 0) M.dps[w.ph][16 * w.it + w.l16] = dps;
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
#pragma unroll
                        for (int q = 0; q < TT; ++q) {
                            const int r0 = 16 * T + 4 * w.g + q * R, tt = r0 / R;   // a token's rows
                            const bool off = tl < tt, on = tl == tt;
                            const float ex = off ? exp2_fast(o.c2[r0] - c2j) : 0.f;
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
                                const float val = od * wt;
                                colc += val;
                                const float rs = sum16(val);
                                if (w.l16 == 0) M.rc[J][r0] = rs;
                            } else {
                                cols += od * ex;
                                if (T == J) {
                                    const float rs = sum16(on ? dW : 0.f);
                                    if (w.l16 == 0) M.rg[r0] = rs;
                                }
                            }
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
#pragma unroll
                        for (int q = 0; q < TT; ++q) {
                            const int r0 = 16 * Jt + 4 * w.g + q * R, tj = r0 / R;
                            const float wt = tj < tl ? exp2_fast(c2t - o.c2[r0]) * o.sig[r0] : tj == tl ? gmt : 0.f;
#pragma unroll
                            for (int r = 0; r < R; ++r) gT[q * R + r] *= wt;
                        }
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) wT[jp][4 * h + v] = (bf16)gT[v];
                }
        }
        if (more) tok_scan<R>(a, w, c - 1, valid(c - 1), raw, M.seg, M.tok[par ^ 1]);
        __syncthreads();

        // ======== region 1: the chunk's gradients ========
        const float vj = o.v[row], ec = o.ec[row];
        const int64_t trow = s.tok + (t0 + tl) * a.H;   // (this lane's token; stored when tl < nvalid)
        const int rk = row % R;
        {
            // dx: columns 32 hf + 8 g + e
            f32x4 d[2], bu[2];
#pragma unroll
            for (int ab = 0; ab < 2; ++ab) {
                d[ab] = bu[ab] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kp = 0; kp < 2; ++kp)
                    if (2 * kp + 1 >= J) d[ab] = MM::mma(perm_kt2(M.Y, LDP, 32 * kp, 32 * hf, ab, w.g, w.l16), wG[kp], d[ab]);
#pragma unroll
                for (int kk = 0; kk < 4; ++kk)
                    bu[ab] = MM::mma(perm_kt(M.U, LDP, 32 * kk, 32 * hf, ab, w.g, w.l16), fB[kk], bu[ab]);
            }
            const bf16x8 xv = MM::load(&M.X[row * LDP + 32 * hf + 8 * w.g]);
            const bf16x8 yv = MM::load(&M.Y[row * LDP + 32 * hf + 8 * w.g]);
            float dvp = 0.f;
            bf16x8 out;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float xe = (float)xv[e], ye = (float)yv[e], be = bu[e / 4][e % 4];
                dvp += xe * be;
                xdy += xe * ye;
                out[e] = (bf16)(d[e / 4][e % 4] + vj * be + Dh * ye);
            }
            if (tl < nvalid)
                *reinterpret_cast<bf16x8 *>(static_cast<bf16 *>(a.dx) + (trow * R + rk) * kP + 32 * hf + 8 * w.g) = out;
            dvp = sum_g(dvp);
            if (w.g == 0) M.dv[hf][row] = dvp;
        }
        float cn[8], sn[8], dpsi[8];
        cs_getn<8>(&cs[tl * kNH + 32 * hf + 8 * w.g], cn, sn);
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
                            d[q][ab] = MM::mma(perm_kt2(M.C, LDN, 32 * kp, 64 * q + 32 * hf, ab, w.g, w.l16), wD[kp], d[q][ab]);
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
                        xu[q][ab] = MM::mma(perm_rows(M.U, LDP, 64 * q + 32 * hf, 32 * kk, ab, w.g, w.l16), fX[kk], xu[q][ab]);
                }
            const bf16x8 br = MM::load(&M.B[row * LDN + 32 * hf + 8 * w.g]);
            const bf16x8 bi = MM::load(&M.B[row * LDN + 64 + 32 * hf + 8 * w.g]);
            bf16x8 o0, o1;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float re = d[0][e / 4][e % 4] + vj * xu[0][e / 4][e % 4];
                const float im = d[1][e / 4][e % 4] + vj * xu[1][e / 4][e % 4];
                dpsi[e] = re * (float)bi[e] - im * (float)br[e];
                o0[e] = (bf16)(cn[e] * re - sn[e] * im);
                o1[e] = (bf16)(sn[e] * re + cn[e] * im);
            }
            if (tl < nvalid) {
                bf16 *p = static_cast<bf16 *>(a.dB) + (trow * R + rk) * kN + 32 * hf + 8 * w.g;
                *reinterpret_cast<bf16x8 *>(p) = o0;
                *reinterpret_cast<bf16x8 *>(p + kNH) = o1;
            }
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
                            d[q][ab] = MM::mma(perm_kt2(M.B, LDN, 32 * jp, 64 * q + 32 * hf, ab, w.g, w.l16), wT[jp], d[q][ab]);
#pragma unroll
                    for (int kk = 0; kk < 2; ++kk)
                        t2[q][ab] = MM::mma(perm_rows(M.S, LDP, 64 * q + 32 * hf, 32 * kk, ab, w.g, w.l16), fY[kk], t2[q][ab]);
                }
            const bf16x8 cr = MM::load(&M.C[row * LDN + 32 * hf + 8 * w.g]);
            const bf16x8 ci = MM::load(&M.C[row * LDN + 64 + 32 * hf + 8 * w.g]);
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
            if (tl < nvalid) {
                bf16 *p = static_cast<bf16 *>(a.dC) + (trow * R + rk) * kN + 32 * hf + 8 * w.g;
                *reinterpret_cast<bf16x8 *>(p) = o0;
                *reinterpret_cast<bf16x8 *>(p + kNH) = o1;
            }
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
        float nx_dt = 0.f, nx_lam = 0.f, nx_A = 0.f;
        if (more) {
            tok_table<R>(w, valid(c - 1), raw, M.seg, M.cs[par ^ 1], M.tok[par ^ 1]);
            nx_dt = raw.dt; nx_lam = raw.lam; nx_A = raw.A;
            if (k + 2 < n) load_tok<R>(a, s, w, c - 2, valid(c - 2), raw);
        }
        __syncthreads();

        // ======== region 2: next rows, dtheta, per-token scalars ========
        if (more) {
            stage(valid(c - 1), M.cs[par ^ 1], M.tok[par ^ 1]);
            if (k + 2 < n) load_rows(c - 2);
        }
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
        __syncthreads();
    }
    if (seg == 0 && a.dinit) store_np(G, a.dinit + bh * kMap, w);
    // per-segment partials of dD and dA
    xdy = sum_wave(xdy);
    if (w.lane == 0) M.red[w.wave] = xdy;
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
    __shared__ float s_a[kThrF], s_d[kThrF];
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
    float sa = 0.f, sd = 0.f;
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
        a.dD[h] = s_d[0];
        if (!a.dA_per_token) a.dA[h] = s_a[0];
    }
}

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
    for (int64_t ns = 1; ns <= most; ++ns) {
        const int64_t G = (nchunks + ns - 1) / ns, m = (nchunks + G - 1) / G;
        double t = (double)((BH * m + ncu - 1) / ncu) * G * kMain;
        if (m > 1) t += (double)((BH * (m - 1) * 2 + 2 * ncu - 1) / (2 * ncu)) * G * kAggr + kPass + kFold * m;
        if (ns == 1 || t < best) {
            best = t;
            bestG = G;
        }
    }
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
    w.off_dsig = up(w.off_tot + segs * 2 * (size_t)(1 + N / 2) * sizeof(float));
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

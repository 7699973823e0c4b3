// Prefill scan by workgroups that walk a segment of a slice's chunks with the
// state in registers: bf16, P = 64, N = 64 or 32, on gfx950.
//
// The decomposition is that of the other prefill kernels (m3_prefill.hip) on
// chunks of 64 rows (64 / R tokens) whatever the caller's chunk: the scan
// does not depend on it, and 64 rows are what one 16-row tile a wave covers.
// A slice's chunks are split into segments, so that the launch fills the
// device:
//   k_walk<false>  only with several segments a slice: the map of every
//                  segment but the last from a zero state (B, x and the
//                  angles read, nothing stored but the map)
//   k_walk_pass    only with many segments a slice: the maps folded over them
//   k_walk<true>   every segment from its entering state (the fold of the maps
//                  before it): y, and from the last one the final state and
//                  carry
// Per chunk: y^T = e^{cum_t} S^T C^_t + x^T (w o G)^T + D x with G^T = B^ C^T
// (MFMA, the output transposed with permuted rows, so that a lane holds eight
// consecutive channels of one row), then S <- R(psi_e)(e^{cum_e} S + (v B^)^T x).
// The next chunk's rows and the angles of the one after are in flight while a
// chunk is worked on; the loads and stores of the loop are unconditional (a
// ragged chunk's spare lanes repeat the last token), so that a wait for loads
// never waits for the stores after them.
//
// Bound: issue and LDS of a CU (a chunk 3.5 us of a CU's time against 1.1 us
// for its bytes), and the second read of B, x and the angles.  Measured on B=4
// L=2000 H=16 N=64 SISO, gated, from a state: 51 us; the three kernels with an
// N x P map stored per chunk, element-wise loads and a sine and cosine per
// element: 163 us (both timed in a loop).  The cosines and sines are held in
// fp32, as those kernels formed them (in fp16 the state is 0.5% further from
// fp64; y 2.87e-3 and state 1.67e-3 are theirs to four digits).
#include <stddef.h>

#include <algorithm>

#include "m3_device.h"
#include "m3_internal.h"
#include "m3_scan_common.h"

namespace m3 {
namespace {

using namespace scan;

constexpr int kRows = 64, kP = 64;
constexpr float kLog2e = 1.44269504088896340736f;
typedef Mma<bf16> MM;
// Segments a slice up to which a workgroup folds the maps before its own by
// itself; more go through k_walk_pass.
constexpr int kFold = 16;

template <int N_, int R_> struct Walk {
    static constexpr int N = N_, R = R_, NH = N / 2;
    static constexpr int NW = 4, NTHR = NW * kWave;
    static constexpr int Q = kRows / R;          // tokens a chunk
    static constexpr int TG = NTHR / NH;         // token groups of the angle scan
    static constexpr int TPS = Q / TG;           // tokens a group
    static constexpr int NIT = N / 32;           // 16-row tiles of rotation pairs
    static constexpr int U = NIT * (kP / 16) / NW;   // (pair tile, column tile) units a wave
    static constexpr int KC = N / 32;            // K steps along the state
    static constexpr int LDN = N + 16, LDP = kP + 16;   // padded LDS rows
    static constexpr int BT = kRows * NH / 8;    // tasks of the B rows (a piece pair each)
    static constexpr int XT = kRows * kP / 8 / NTHR;   // x pieces a thread
    // LDS besides the cos / sin table, and the workgroups of a CU with rows of
    // `w` pairs in that (the LDS is given out in pieces of 2 KB)
    static constexpr int kFixed = 2 * kRows * LDN * 2 + kRows * LDP * 2 + kP * LDN * 2 + NTHR * 4 +
                                  3 * (3 * kRows + 2 * NH) * 4;
    static constexpr int per_cu(int w) { return 160 * 1024 / ((kFixed + Q * w * 8 + 2047) / 2048 * 2048); }
    static constexpr bool kPadCs = per_cu(NH + 2) == per_cu(NH);
    static constexpr int LDC = kPadCs ? NH + 2 : NH;
    static constexpr int kMap = N * kP, kTot = 2 * NH + 4;   // floats of a segment's map and totals
    static_assert(kTot * 4 <= kMap * 2, "the totals of a segment fit a chunk's share of Sin");
    static_assert(Q % TG == 0 && U >= 1 && BT <= NTHR, "work split");
};

// A chunk's scalars by row (token, rank): base-2 log-decay prefix, gamma,
// sigma (rows past the end: the total decay, so that c2[kRows - 1] always is it,
// and zeros); the cosines and sines of the pairs' total angles.
template <class W> struct alignas(16) WTok {
    float c2[kRows], gam[kRows], sig[kRows];
    float ce[W::NH], se[W::NH];
};
// (the tables are read in 16-byte pieces, in every slot of an array)
template <class T> constexpr bool tok_aligned() {
    return sizeof(T) % 16 == 0 && offsetof(T, c2) % 16 == 0 && offsetof(T, sig) % 16 == 0 &&
           offsetof(T, ce) % 16 == 0 && offsetof(T, se) % 16 == 0;
}

template <class W> struct alignas(16) WLds {
    bf16 B[kRows * W::LDN];     // B^ rows, and v B^ (scaled before its one rounding)
    bf16 VB[kRows * W::LDN];
    bf16 X[kRows * W::LDP];     // x rows, channels in tile order (chan_at)
    bf16 S[kP * W::LDN];        // S^T entering the chunk [p in tile order][n]
    float2 cs[W::Q * W::LDC];   // cosine and sine of psi_t, in the order of cs_unit
    float seg[W::TG][W::NH];
    WTok<W> tok[3];
};

// Two pairs' entries (16 bytes, unit u of a row's NH / 2) of the table's row t.
// Rows padded by 16 bytes let 16 lanes read one unit of 16 rows, or four units
// of four rows, from different banks.  Where the padding would cost a CU a
// workgroup (N = 64 at rank 2, N = 32 at rank 1: 15% on B=155 L=363 H=8), the units
// of a row are exchanged by its number instead (the address takes 2% more time).
template <class W> __device__ __forceinline__ int cs_unit(int t, int u) {
    constexpr int UN = W::NH / 2;
    return t * W::LDC + 2 * (W::kPadCs ? u : u ^ (t / (16 / UN) % UN));
}
template <class W> __device__ __forceinline__ void cs_get8(const float2 *cs, int t, int i, float (&c)[8], float (&s)[8]) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const f32x4 w = *reinterpret_cast<const f32x4 *>(&cs[cs_unit<W>(t, i / 2 + j)]);
        c[2 * j] = w[0];
        s[2 * j] = w[1];
        c[2 * j + 1] = w[2];
        s[2 * j + 1] = w[3];
    }
}

struct WAt {   // the slice's offsets
    int64_t b, h, tok, L, H;
};

// Offset that takes a pointer at token t of a chunk back to its last valid
// token when t is past the end (only the sequence's last chunk is ragged, so
// the branch is uniform and rarely taken).
__device__ __forceinline__ int64_t past_end(int t, int nvalid, int q, int64_t stride) {
    int64_t o = 0;
    if (nvalid < q) {
        asm volatile("");   // (a branch, not selects on every load)
        o = t >= nvalid ? (nvalid - 1 - t) * stride : 0;
    }
    return o;
}

// Loads run a chunk ahead of their use: each thread holds 64-bit pointers to
// its place in the chunk to be loaded next, advanced by one chunk at a time
// (no per-load address products, no limit on the token stride).
template <class W> struct WCur {
    const float *th;       // angles of its first token and pair (omega: M3_THETA_PER_HEAD)
    const bf16 *b, *x;     // B and x pieces (x: further ones 32 rows apart)
    const bf16 *c, *z;     // C row and gate row of its output lane
    int64_t ct;            // the chunk's first token
    int64_t sth, sb, sx;   // strides of a token, in elements
};

// Raw values of a chunk's prologue: angles of the thread's tokens; by wave 0,
// one lane a row, the token's scalars.
template <class W> struct WRaw {
    float th[W::TPS], dts[W::TPS];
    float dt, lam, A, dtn, lamn;
};
template <class W> struct WRows {   // a chunk's B and x pieces as this thread stages them
    bf16x8 lo, hi, x[W::XT];
};
// The C row of output lane (row, g) as MFMA fragments; N = 32 keeps the
// partner half of each pair beside it (it lies in another lane).
template <class W> struct WC {
    bf16x8 f[W::KC], o;
};

template <class W>
__device__ __forceinline__ void load_tok(const ScanArgs &a, const WAt &s, int tid, const WCur<W> &u, int nvalid, WRaw<W> &r) {
    const int tg = tid / W::NH;
#pragma unroll
    for (int k = 0; k < W::TPS; ++k)
        r.th[k] = u.th[k * u.sth + past_end(tg * W::TPS + k, nvalid, W::Q, u.sth)];
    if (a.theta_ph) {
#pragma unroll
        for (int k = 0; k < W::TPS; ++k)
            r.dts[k] = a.dt[s.tok + (u.ct + min(tg * W::TPS + k, nvalid - 1)) * s.H];
    }
    if (__builtin_amdgcn_readfirstlane(tid) < kWave) {
        const int64_t t = u.ct + min((tid & (kWave - 1)) / W::R, nvalid - 1), tn = min(t + 1, s.L - 1);
        r.dt = a.dt[s.tok + t * s.H];
        r.lam = a.lam[s.tok + t * s.H];
        r.A = a.A[s.b * a.a_sb + t * a.a_st + s.h * a.a_sh];
        r.dtn = a.dt[s.tok + tn * s.H];
        r.lamn = a.lam[s.tok + tn * s.H];
    }
}
template <class W>
__device__ __forceinline__ void load_rows(int tid, const WCur<W> &u, int nvalid, WRows<W> &r) {
    // (threads past the B tasks repeat the last one's load)
    const bf16 *p = u.b + past_end(min(tid, W::BT - 1) / (W::NH / 8) / W::R, nvalid, W::Q, u.sb);
    r.lo = *reinterpret_cast<const bf16x8 *>(p);
    r.hi = *reinterpret_cast<const bf16x8 *>(p + W::NH);
#pragma unroll
    for (int k = 0; k < W::XT; ++k) {
        const int t = (tid + k * W::NTHR) / 8 / W::R;
        r.x[k] = *reinterpret_cast<const bf16x8 *>(u.x + k * (W::NTHR / 8 / W::R) * u.sx + past_end(t, nvalid, W::Q, u.sx));
    }
}
template <class W>
__device__ __forceinline__ void load_c(int t, int g, const WCur<W> &u, int nvalid, WC<W> &r) {
    const bf16 *p = u.c + past_end(t, nvalid, W::Q, u.sb);
#pragma unroll
    for (int kk = 0; kk < W::KC; ++kk) r.f[kk] = *reinterpret_cast<const bf16x8 *>(p + kk * 32);
    if constexpr (W::N == 32) r.o = *reinterpret_cast<const bf16x8 *>(p + (g < 2 ? 16 : -16));
}

// The threads' angle prefix sums over their tokens (the group's total to
// `seg`), and by wave 0 the scalar tables.  Tokens past the end get zero
// angles and weights.
template <class W>
__device__ __forceinline__ void tok_scan(const ScanArgs &a, const WAt &s, int tid, int64_t ct, int nvalid,
                                         const WRaw<W> &r, float (&ps)[W::TPS], WLds<W> &L, WTok<W> &o) {
    const int i = tid % W::NH, tg = tid / W::NH;
#pragma unroll
    for (int k = 0; k < W::TPS; ++k) ps[k] = r.th[k];
    if (a.theta_ph) {
#pragma unroll
        for (int k = 0; k < W::TPS; ++k) ps[k] *= r.dts[k];
    }
    if (nvalid < W::Q) {
#pragma unroll
        for (int k = 0; k < W::TPS; ++k) ps[k] = tg * W::TPS + k < nvalid ? ps[k] : 0.f;
    }
#pragma unroll
    for (int k = 1; k < W::TPS; ++k) ps[k] += ps[k - 1];
    L.seg[tg][i] = ps[W::TPS - 1];
    if (__builtin_amdgcn_readfirstlane(tid) < kWave) {
        const int t = tid / W::R;
        const bool in = t < nvalid;
        const float c2 = lane_scan(in && tid % W::R == 0 ? r.dt * r.A * kLog2e : 0.f);
        const float c2e = lane_bcast(c2, nvalid * W::R - 1);
        const float gam = in ? r.lam * r.dt : 0.f;
        float sig = gam;
        if (in && ct + t + 1 < s.L) sig += (1.f - r.lamn) * r.dtn;
        o.c2[tid] = in ? c2 : c2e;
        o.gam[tid] = gam;
        o.sig[tid] = sig;
    }
}

// The cos / sin table of psi_t, in fp32, and that of psi_e, which turns the
// state in every chunk, to the last bit.  Returns psi_e of its pair in the
// threads that hold the last token.
template <class W>
__device__ __forceinline__ float tok_table(int tid, int nvalid, const float (&ps)[W::TPS], WLds<W> &L, WTok<W> &o) {
    const int i = tid % W::NH, tg = tid / W::NH;
    float off = 0.f;
#pragma unroll
    for (int q = 0; q < W::TG - 1; ++q) off += q < tg ? L.seg[q][i] : 0.f;
    float pe = 0.f;
#pragma unroll
    for (int k = 0; k < W::TPS; ++k) {
        const float psi = ps[k] + off;
        float sn, cn;
        sincos_rev(psi, &sn, &cn);
        L.cs[cs_unit<W>(tg * W::TPS + k, i / 2) + i % 2] = make_float2(cn, sn);
        if (k == (nvalid - 1) % W::TPS) pe = psi;
    }
    if (tg == (nvalid - 1) / W::TPS) sincos_full(pe, &o.se[i], &o.ce[i]);
    return pe;
}

template <class W, bool kOut>
__device__ __forceinline__ void stage(int tid, int nvalid, WRows<W> &r, WLds<W> &L, const WTok<W> &o) {
    if (nvalid < W::Q) {   // rows past the end are zero
        const bf16x8 z = {};
        if (tid / (W::NH / 8) / W::R >= nvalid) r.lo = r.hi = z;
#pragma unroll
        for (int k = 0; k < W::XT; ++k)
            if ((tid + k * W::NTHR) / 8 / W::R >= nvalid) r.x[k] = z;
    }
    if (W::BT == W::NTHR || tid < W::BT) {
        const int row = tid / (W::NH / 8), cp = tid % (W::NH / 8);
        const float v = exp2_fast(o.c2[kRows - 1] - o.c2[row]) * o.sig[row];
        float c[8], sn[8];
        cs_get8<W>(L.cs, row / W::R, cp * 8, c, sn);
        bf16x8 lo, hi, vlo, vhi;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float u = (float)r.lo[e], x = (float)r.hi[e];
            const float re = c[e] * u + sn[e] * x, im = c[e] * x - sn[e] * u;
            lo[e] = (bf16)re;
            hi[e] = (bf16)im;
            vlo[e] = (bf16)(v * re);
            vhi[e] = (bf16)(v * im);
        }
        if constexpr (kOut) {
            *reinterpret_cast<bf16x8 *>(&L.B[row * W::LDN + cp * 8]) = lo;
            *reinterpret_cast<bf16x8 *>(&L.B[row * W::LDN + W::NH + cp * 8]) = hi;
        }
        *reinterpret_cast<bf16x8 *>(&L.VB[row * W::LDN + cp * 8]) = vlo;
        *reinterpret_cast<bf16x8 *>(&L.VB[row * W::LDN + W::NH + cp * 8]) = vhi;
    }
#pragma unroll
    for (int k = 0; k < W::XT; ++k) {
        const int row = (tid + k * W::NTHR) / 8, cp = tid % 8;
        put_tile_order(&L.X[row * W::LDP], cp, r.x[k]);
    }
}

template <class W>
__device__ __forceinline__ void rotate_c(WC<W> &r, const float2 *cs, int t, int g) {
    if constexpr (W::N == 32) {
        float c[8], sn[8];
        cs_get8<W>(cs, t, 8 * (g & 1), c, sn);
        const float sg = g < 2 ? 1.f : -1.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) r.f[0][e] = (bf16)(c[e] * (float)r.f[0][e] + sg * sn[e] * (float)r.o[e]);
    } else {
#pragma unroll
        for (int kk = 0; kk < W::KC / 2; ++kk) {
            float c[8], sn[8];
            cs_get8<W>(cs, t, kk * 32 + 8 * g, c, sn);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float u = (float)r.f[kk][e], v = (float)r.f[kk + W::KC / 2][e];
                r.f[kk][e] = (bf16)(c[e] * u + sn[e] * v);
                r.f[kk + W::KC / 2][e] = (bf16)(c[e] * v - sn[e] * u);
            }
        }
    }
}

// The state after `n` segments of a slice whose maps start at `slot`, from the
// state `st` before them: S <- e^{sum cum} R(sum psi) S + map; `after` is
// called with each segment's slot once its step is done.  A segment's totals
// (kTot floats of the workspace's Sin): the cosines and sines of its pairs'
// angles, and its log-decay (base 2).
template <class W, class F>
__device__ __forceinline__ void fold(const ScanArgs &a, int64_t slot, int n, int it, int g, int tid,
                                     f32x4 (&st)[2][W::U], F after) {
    constexpr int DEPTH = 4;   // segments whose loads are issued together
    for (int k0 = 0; k0 < n; k0 += DEPTH) {
        f32x4 m[DEPTH][2][W::U], cn[DEPTH], sn[DEPTH];
        float c2[DEPTH];
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int64_t k = slot + min(k0 + d, n - 1);
            const float *tot = static_cast<const float *>(a.Sin) + k * W::kTot;
            cn[d] = *reinterpret_cast<const f32x4 *>(&tot[16 * it + 4 * g]);
            sn[d] = *reinterpret_cast<const f32x4 *>(&tot[W::NH + 16 * it + 4 * g]);
            c2[d] = tot[2 * W::NH];
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int u = 0; u < W::U; ++u)
                    m[d][q][u] = *reinterpret_cast<const f32x4 *>(&a.M[k * W::kMap + ((q * W::U + u) * W::NTHR + tid) * 4]);
        }
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            if (k0 + d >= n) break;
            const float e = exp2_fast(c2[d]);
#pragma unroll
            for (int u = 0; u < W::U; ++u) {
                const f32x4 re = st[0][u], im = st[1][u];
                st[0][u] = e * (cn[d] * re - sn[d] * im) + m[d][0][u];
                st[1][u] = e * (sn[d] * re + cn[d] * im) + m[d][1][u];
            }
            after(slot + k0 + d);
        }
    }
}

// ---------------------------------------------------------------------------
// k_walk: grid (slices, segments), one segment a workgroup.  State element
// (unit u, half q, v): row n = q N/2 + 16 it + 4 g + v, column p = the channel at
// tile position 16 (pt + u) + l16 (chan_of).
// ---------------------------------------------------------------------------
template <int N, int R, bool kOut, bool kGate>
__global__ __launch_bounds__(256, 2) void k_walk(ScanArgs a) {
    typedef Walk<N, R> W;
    static_assert(tok_aligned<WTok<W>>() && offsetof(WLds<W>, tok) % 16 == 0 && offsetof(WLds<W>, cs) % 16 == 0,
                  "16-byte pieces");
    static_assert(sizeof(WLds<W>) == W::kFixed + W::Q * W::LDC * 8, "LDS as counted");
    __shared__ WLds<W> L;
    int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int64_t bh = blockIdx.x, seg = blockIdx.y;
    const WAt s = {bh / a.H, bh % a.H, bh / a.H * a.L * a.H + bh % a.H, a.L, a.H};
    const int64_t n64 = (a.L + W::Q - 1) / W::Q;
    const int64_t c0 = seg * a.G, n = min(a.G, n64 - c0);
    const int it = wave % W::NIT, pt = wave / W::NIT * W::U;
    auto valid = [&](int64_t c) { return (int)min((int64_t)W::Q, a.L - c * W::Q); };

    f32x4 st[2][W::U];
    const float Dh = a.D[s.h];
    WCur<W> u;
    u.ct = c0 * W::Q;
    u.sth = a.theta_ph ? 0 : s.H * W::NH;
    u.sb = s.H * R * N;
    u.sx = s.H * R * kP;
    int64_t ycur;   // y (and gate) element of the output lane in the chunk worked on
    {
        const int lane = tid & (kWave - 1), g = lane >> 4, row = 16 * wave + (lane & 15);
        const int64_t at = s.tok + u.ct * s.H;
        u.th = a.theta + (a.theta_ph ? s.h * W::NH : at * W::NH) + tid / W::NH * W::TPS * u.sth + tid % W::NH;
        const int bt = min(tid, W::BT - 1), br = bt / (W::NH / 8);
        u.b = static_cast<const bf16 *>(a.B) + at * (R * N) + br / R * u.sb + br % R * N + bt % (W::NH / 8) * 8;
        u.x = static_cast<const bf16 *>(a.x) + at * (R * kP) + tid / 8 / R * u.sx + tid / 8 % R * kP + tid % 8 * 8;
        u.c = static_cast<const bf16 *>(a.C) + at * (R * N) + row / R * u.sb + row % R * N + 8 * g;
        ycur = at * (R * kP) + row / R * u.sx + row % R * kP + 8 * g;
        u.z = static_cast<const bf16 *>(a.z) + ycur;
    }
    WRaw<W> raw;
    WRows<W> rows;
    WC<W> cf, cn;
    bf16x8 zr[2], zn[2];
    float ps[W::TPS];
    // (maps: the segment's totals, thousands of radians in a long one; its chunks
    // are whole, so the last threads hold every psi_e)
    double psum = 0.0, c2sum = 0.0;
    auto put_state = [&](int lane) {
        const int g = lane >> 4, l16 = lane & 15;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < W::U; ++v)
                store4(&L.S[(16 * (pt + v) + l16) * W::LDN + q * W::NH + 16 * it + 4 * g], st[q][v]);
    };
    // the loads of chunk c's rows, C and gate (which the cursors stand at),
    // then the cursors to chunk c + 1 (kept at the segment's last chunk)
    auto fetch = [&](int64_t c) {
        const int nv = valid(c), lane = tid & (kWave - 1), g = lane >> 4, t = (16 * wave + (lane & 15)) / R;
        load_rows<W>(tid, u, nv, rows);
        if constexpr (kOut) {
            load_c<W>(t, g, u, nv, cn);
            if constexpr (kGate) {
                const bf16 *z = u.z + past_end(t, nv, W::Q, u.sx);
                zn[0] = *reinterpret_cast<const bf16x8 *>(z);
                zn[1] = *reinterpret_cast<const bf16x8 *>(z + 32);
            }
        }
        const int64_t q = c + 1 < c0 + n ? W::Q : 0;
        u.b += q * u.sb;
        u.x += q * u.sx;
        u.c += q * u.sb;
        u.z += q * u.sx;
    };
    auto fetch_tok = [&](int64_t c) {
        load_tok<W>(a, s, tid, u, valid(c), raw);
        const int64_t q = c + 1 < c0 + n ? W::Q : 0;
        u.th += q * u.sth;
        u.ct += q;
    };
    const int64_t ce = c0 + n - 1;
    if (n > 0) {
        fetch_tok(c0);
        fetch(c0);
    }
    // entering state (a map starts from zero)
    {
        const int lane = tid & (kWave - 1), g = lane >> 4, l16 = lane & 15;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int v = 0; v < W::U; ++v) st[q][v] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (kOut && (seg == 0 || a.nseg <= kFold)) {
            float el[2 * W::U * 4];
            const bool carry = a.init_cB && a.L > 0;
            init_elems<bf16, R, N, kP, 2 * W::U * 4>(
                a.init_state ? a.init_state + bh * W::kMap : nullptr,
                carry ? static_cast<const bf16 *>(a.init_cB) + bh * (R * N) : nullptr,
                carry ? static_cast<const bf16 *>(a.init_cX) + bh * (R * kP) : nullptr,
                a.L > 0 ? (1.f - a.lam[s.tok]) * a.dt[s.tok] : 0.f,
                [&](int k) { return k / (4 * W::U) * W::NH + 16 * it + 4 * g + k % 4; },
                [&](int k) { return chan_of(16 * (pt + k / 4 % W::U) + l16); }, el);
#pragma unroll
            for (int k = 0; k < 2 * W::U * 4; ++k) st[k / (4 * W::U)][k / 4 % W::U][k % 4] = el[k];
            fold<W>(a, bh * a.nseg, (int)seg, it, g, tid, st, [](int64_t) {});
        } else if (kOut) {
            const float *m = a.M + (bh * a.nseg + seg - 1) * W::kMap;
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < W::U; ++v)
                    st[q][v] = *reinterpret_cast<const f32x4 *>(&m[((q * W::U + v) * W::NTHR + tid) * 4]);
        }
    }
    if (n > 0) {
        const int64_t c1 = min(c0 + 1, ce), c2 = min(c0 + 2, ce);
        const int lane = tid & (kWave - 1), g = lane >> 4, t = (16 * wave + (lane & 15)) / R;
        tok_scan<W>(a, s, tid, c0 * W::Q, valid(c0), raw, ps, L, L.tok[0]);
        fetch_tok(c1);
        __syncthreads();
        psum = tok_table<W>(tid, valid(c0), ps, L, L.tok[0]);
        __syncthreads();
        stage<W, kOut>(tid, valid(c0), rows, L, L.tok[0]);
        if constexpr (kOut) {
            cf = cn;
            zr[0] = zn[0];
            zr[1] = zn[1];
            rotate_c<W>(cf, L.cs, min(t, valid(c0) - 1), g);
            put_state(lane);
        }
        fetch(c1);
        tok_scan<W>(a, s, tid, c1 * W::Q, valid(c1), raw, ps, L, L.tok[1]);
        fetch_tok(c2);
        __syncthreads();
    }
    int p0 = 0, p1 = 1, p2 = 2;   // scalar tables of chunks c, c + 1, c + 2
    for (int64_t c = c0; c <= ce; ++c) {
        const int64_t c1 = min(c + 1, ce), c2 = min(c + 2, ce), c3 = min(c + 3, ce);   // (past the end: loaded unused)
        const int nvalid = valid(c), nv1 = valid(c1);
        const WTok<W> &o = L.tok[p0];
        asm volatile("" : "+v"(tid));   // (no address held in registers across the loop)
        const int lane = tid & (kWave - 1), g = lane >> 4, l16 = lane & 15;
        // ======== y of chunk c, the state after it; the table of chunk c + 1 ========
        if constexpr (kOut) {
            // (lanes past the end of the sequence repeat the last token's
            // row, weights and store: the stores need no mask)
            const int tl = min((16 * wave + l16) / R, nvalid - 1), row = tl * R + l16 % R;
            f32x4 y[2][2];
#pragma unroll
            for (int hp = 0; hp < 2; ++hp)
#pragma unroll
                for (int ab = 0; ab < 2; ++ab) {
                    y[hp][ab] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kk = 0; kk < W::KC; ++kk)
                        y[hp][ab] = MM::mma(MM::load(&L.S[(32 * hp + 16 * ab + l16) * W::LDN + 32 * kk + 8 * g]), cf.f[kk], y[hp][ab]);
                }
            const float c2t = o.c2[row], gmt = o.gam[row], ec = exp2_fast(c2t);
#pragma unroll
            for (int hp = 0; hp < 2; ++hp)
#pragma unroll
                for (int ab = 0; ab < 2; ++ab) y[hp][ab] *= ec;
#pragma unroll
            for (int jp = 0; jp < 2; ++jp) {
                if (2 * jp > wave) continue;
                bf16x8 wt;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int J = 2 * jp + h;
                    f32x4 gt = {0.f, 0.f, 0.f, 0.f};
                    if (J <= wave) {
#pragma unroll
                        for (int kk = 0; kk < W::KC; ++kk)
                            gt = MM::mma(MM::load(&L.B[(16 * J + l16) * W::LDN + 32 * kk + 8 * g]), cf.f[kk], gt);
                        const f32x4 c4 = *reinterpret_cast<const f32x4 *>(&o.c2[16 * J + 4 * g]);
                        const f32x4 s4 = *reinterpret_cast<const f32x4 *>(&o.sig[16 * J + 4 * g]);
#pragma unroll
                        for (int q = 0; q < 4; q += R) {
                            const int tj = (16 * J + 4 * g + q) / R;
                            // (no token of an earlier tile is past the lane's own, unless the
                            // lane repeats an earlier row)
                            float w = tj < tl ? exp2_fast(c2t - c4[q]) * s4[q] : 0.f;
                            w = tj == tl ? gmt : w;
#pragma unroll
                            for (int r = 0; r < R; ++r) gt[q + r] *= w;
                        }
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) wt[4 * h + v] = (bf16)gt[v];
                }
#pragma unroll
                for (int hp = 0; hp < 2; ++hp)
#pragma unroll
                    for (int ab = 0; ab < 2; ++ab)
                        y[hp][ab] = MM::mma(load_kt2(L.X, W::LDP, 32 * jp, 32 * hp + 16 * ab, g, l16), wt, y[hp][ab]);
            }
            bf16 *yp = static_cast<bf16 *>(a.y) + ycur + past_end((16 * wave + l16) / R, nvalid, W::Q, u.sx);
#pragma unroll
            for (int hp = 0; hp < 2; ++hp) {
                const bf16x8 xv = get_tile_order(&L.X[row * W::LDP], 4 * hp + g);
                bf16x8 out;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    float v = y[hp][e / 4][e % 4] + Dh * (float)xv[e];
                    if constexpr (kGate) v *= silu((float)zr[hp][e]);
                    out[e] = (bf16)v;
                }
                *reinterpret_cast<bf16x8 *>(yp + 32 * hp) = out;
            }
            ycur += W::Q * u.sx;
        }
        {
            const float e = exp2_fast(o.c2[kRows - 1]);
#pragma unroll
            for (int q = 0; q < 2; ++q)
#pragma unroll
                for (int v = 0; v < W::U; ++v) st[q][v] *= e;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                bf16x8 xc[W::U];
#pragma unroll
                for (int v = 0; v < W::U; ++v) xc[v] = load_kt(L.X, W::LDP, 32 * ks, 16 * (pt + v), g, l16);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const bf16x8 bn = load_kt(L.VB, W::LDN, 32 * ks, q * W::NH + 16 * it, g, l16);
#pragma unroll
                    for (int v = 0; v < W::U; ++v) st[q][v] = MM::mma(bn, xc[v], st[q][v]);
                }
            }
            const f32x4 cn4 = *reinterpret_cast<const f32x4 *>(&o.ce[16 * it + 4 * g]);
            const f32x4 sn4 = *reinterpret_cast<const f32x4 *>(&o.se[16 * it + 4 * g]);
#pragma unroll
            for (int v = 0; v < W::U; ++v) {
                const f32x4 re = st[0][v], im = st[1][v];
                st[0][v] = cn4 * re - sn4 * im;
                st[1][v] = sn4 * re + cn4 * im;
            }
            if constexpr (!kOut) c2sum += o.c2[kRows - 1];
        }
        const float pe1 = tok_table<W>(tid, nv1, ps, L, L.tok[p1]);
        if (!kOut && c < ce) psum += pe1;
        __syncthreads();
        // ======== chunk c + 1's rows, C and state; the scans of chunk c + 2 ========
        if constexpr (kOut) {
            put_state(lane);
            cf = cn;
            zr[0] = zn[0];
            zr[1] = zn[1];
            rotate_c<W>(cf, L.cs, min((16 * wave + l16) / R, nv1 - 1), g);
        }
        stage<W, kOut>(tid, nv1, rows, L, L.tok[p1]);
        fetch(c2);
        tok_scan<W>(a, s, tid, c2 * W::Q, valid(c2), raw, ps, L, L.tok[p2]);
        fetch_tok(c3);
        const int p = p0;
        p0 = p1;
        p1 = p2;
        p2 = p;
        __syncthreads();
    }
    if constexpr (!kOut) {
        float *m = a.M + (bh * a.nseg + seg) * W::kMap;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int u = 0; u < W::U; ++u)
                *reinterpret_cast<f32x4 *>(&m[((q * W::U + u) * W::NTHR + tid) * 4]) = st[q][u];
        float *tot = static_cast<float *>(a.Sin) + (bh * a.nseg + seg) * W::kTot;
        if (tid >= W::NTHR - W::NH) {
            float sn, cn;
            sincos_sum(psum, &sn, &cn);
            tot[tid % W::NH] = cn;
            tot[W::NH + tid % W::NH] = sn;
        }
        if (tid == 0) tot[2 * W::NH] = (float)c2sum;
    } else if (seg == a.nseg - 1) {
        const int lane = tid & (kWave - 1), g = lane >> 4, l16 = lane & 15;
        float *fs = a.final_state + bh * W::kMap;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int u = 0; u < W::U; ++u)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    fs[(q * W::NH + 16 * it + 4 * g + v) * kP + chan_of(16 * (pt + u) + l16)] = st[q][u][v];
        // the carry: the last token's B and x (the initial carry of an empty sequence)
        const int64_t last = s.tok + (a.L - 1) * a.H;
        const bf16 *sB = a.L > 0 ? static_cast<const bf16 *>(a.B) + last * (R * N)
                                 : a.init_cB ? static_cast<const bf16 *>(a.init_cB) + bh * (R * N) : nullptr;
        const bf16 *sX = a.L > 0 ? static_cast<const bf16 *>(a.x) + last * (R * kP)
                                 : a.init_cX ? static_cast<const bf16 *>(a.init_cX) + bh * (R * kP) : nullptr;
        bf16 *cB = static_cast<bf16 *>(a.cB) + bh * (R * N), *cX = static_cast<bf16 *>(a.cX) + bh * (R * kP);
        for (int e = tid; e < R * N; e += W::NTHR) cB[e] = sB ? sB[e] : (bf16)0.f;
        for (int e = tid; e < R * kP; e += W::NTHR) cX[e] = sX ? sX[e] : (bf16)0.f;
    }
}

// ---------------------------------------------------------------------------
// k_walk_pass: grid (slices), slices of more than kFold segments: map s
// becomes the state after segment s.
// ---------------------------------------------------------------------------
template <int N, int R>
__global__ __launch_bounds__(256) void k_walk_pass(ScanArgs a) {
    typedef Walk<N, R> W;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave, g = lane >> 4, l16 = lane & 15;
    const int it = wave % W::NIT, pt = wave / W::NIT * W::U;
    const int64_t bh = blockIdx.x, tok = bh / a.H * a.L * a.H + bh % a.H;
    f32x4 st[2][W::U];
    float el[2 * W::U * 4];
    init_elems<bf16, R, N, kP, 2 * W::U * 4>(
        a.init_state ? a.init_state + bh * W::kMap : nullptr,
        a.init_cB ? static_cast<const bf16 *>(a.init_cB) + bh * (R * N) : nullptr,
        a.init_cB ? static_cast<const bf16 *>(a.init_cX) + bh * (R * kP) : nullptr,
        (1.f - a.lam[tok]) * a.dt[tok], [&](int k) { return k / (4 * W::U) * W::NH + 16 * it + 4 * g + k % 4; },
        [&](int k) { return chan_of(16 * (pt + k / 4 % W::U) + l16); }, el);
#pragma unroll
    for (int k = 0; k < 2 * W::U * 4; ++k) st[k / (4 * W::U)][k / 4 % W::U][k % 4] = el[k];
    fold<W>(a, bh * a.nseg, (int)a.nseg - 1, it, g, tid, st, [&](int64_t k) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int u = 0; u < W::U; ++u)
                *reinterpret_cast<f32x4 *>(&a.M[k * W::kMap + ((q * W::U + u) * W::NTHR + tid) * 4]) = st[q][u];
    });
}

// Chunks per segment: the least estimated time over the segment counts (at
// most the caller's chunk count, which sizes the workspace's map area).  From
// B=4 L=2000 H=16 N=64 with 1 to 32 chunks a segment: a chunk takes kChunk in
// a workgroup that has its CU to itself, and 0.87 of that for each of several
// on it (a CU's issue slots and LDS are then full); a map's chunk kMapChunk;
// a workgroup kStart besides, and kFoldStep for each map it folds.
// (4 chunks a segment: 54 us; 3: 58; 8: 63; 32, one segment: 132, with the
// table still in fp16.)
int64_t walk_chunks(int64_t BH, int64_t n64, int64_t most, int64_t ncu) {
    constexpr double kChunk = 4.1, kMapChunk = 2.5, kStart = 5.0, kFoldStep = 0.3;   // us
    double best = 0.0;
    int64_t bestG = n64;
    for_segment_counts(std::min<int64_t>(most, 256), BH, ncu, [&](int64_t ns) {
        const int64_t G = (n64 + ns - 1) / ns, m = (n64 + G - 1) / G;
        auto load = [&](int64_t wgs) { return std::max(1.0, 0.87 * (double)((wgs + ncu - 1) / ncu)); };
        double t = G * kChunk * load(BH * m) + kStart;
        if (m > 1) t += G * kMapChunk * load(BH * (m - 1)) + kStart + kFoldStep * m;
        if (ns == 1 || t < best) {
            best = t;
            bestG = G;
        }
    });
    return bestG;
}

template <int N, int R>
hipError_t launch_walk(const ScanArgs &args, hipStream_t stream) {
    typedef Walk<N, R> W;
    static int cus[64];
    ScanArgs a = args;
    const int64_t BH = a.batch * a.H, n64 = (a.L + W::Q - 1) / W::Q;
    a.G = 1;
    a.nseg = 1;
    if (n64 > 0) {
        const int ncu = cu_count(cus);
        if (ncu <= 0) return hipErrorInvalidDevice;
        a.G = walk_chunks(BH, n64, a.nchunks, ncu);
        a.nseg = (n64 + a.G - 1) / a.G;
    }
    const unsigned nsl = (unsigned)BH, ns = (unsigned)a.nseg;
    if (ns > 1) {
        hipLaunchKernelGGL((k_walk<N, R, false, false>), dim3(nsl, ns - 1), dim3(W::NTHR), 0, stream, a);
        if (ns > kFold) hipLaunchKernelGGL((k_walk_pass<N, R>), dim3(nsl), dim3(W::NTHR), 0, stream, a);
    }
    if (a.z) hipLaunchKernelGGL((k_walk<N, R, true, true>), dim3(nsl, ns), dim3(W::NTHR), 0, stream, a);
    else hipLaunchKernelGGL((k_walk<N, R, true, false>), dim3(nsl, ns), dim3(W::NTHR), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

// bf16, P = 64, the smaller states: every (rank, chunk) the caller may ask
// for (the kernels' own chunk is 64 rows).
ScanImpl find_walk_impl(int io, int64_t N, int64_t P, int64_t R, int64_t Q) {
    const ScanImpl none{nullptr, 0, false, nullptr};
    if (io != 1 || P != kP || R * Q < kRows || R * Q > (N == 64 ? 128 : 64) || R * Q % kRows) return none;
#define M3_CASE(N_, R_) \
    if (N == N_ && R == R_) return ScanImpl{&launch_walk<N_, R_>, (int)sizeof(float), false, nullptr};
    M3_CASE(64, 1) M3_CASE(64, 2) M3_CASE(64, 4) M3_CASE(32, 1) M3_CASE(32, 2) M3_CASE(32, 4)
#undef M3_CASE
    return none;
}

}  // namespace m3

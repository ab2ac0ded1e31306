// Unfused SSD forward: one kernel per step of the block decomposition
// (Section 6), each contraction on the matrix cores.
//
//   k_chunk_prep    step 1: a = dt*A, chunk-local inclusive cumsum (log2 units),
//                           per-chunk scan coefficients (with sequence resets)
//   k_gram          C B^T per (batch, chunk, group), lower block triangle
//   k_chunk_state   right factors: chunk-final states from a zero start
//   k_varlen_final  packed rows: final states of sequences ending inside a chunk
//   k_state_scan    centre factors: scalar SSM scan over chunks, one thread per
//                   (batch, head, p, n) channel (Appendix B sequential mode)
//   k_chunk_output  diagonal block (L o C B^T) X plus left factors C h exp(cs)
//                   plus D x, stored in the activation dtype
//
// Conventions.  cs is in log2 units: cs2_t = log2(e) * sum_{k<=t} dt_k A within
// the chunk, so the 1-SS mask entry L_ts = exp(sum_{s<k<=t} a_k) is
// exp2(cs2_t - cs2_s).  A packed row splits a chunk into segments (maximal runs
// of one sequence id).  A segment "continues" when it starts at the chunk's
// first token and its sequence already ran in the previous chunk (or the chunk
// is the row's first); its incoming state is the state entering the chunk.
// Any other segment starts a sequence; its incoming state is that sequence's
// initial state, decayed from the segment start.
#include "ssd_device.h"
#include "ssd_internal.h"

namespace ssd {
namespace {

constexpr int kThreads = 256;  // 4 wavefronts
constexpr int kMaxQ = 256;
constexpr int kSlab = 64;      // tokens of x (and B) staged in LDS at a time
constexpr int kNB = 64;        // state columns staged in LDS at a time

// Sequence ids outside [0, nseq) break the seq_idx contract; state reads and
// writes for them are skipped so that such input cannot fault the device.
__device__ __forceinline__ bool unit_ok(const Params& p, int64_t u)
{
    return u >= 0 && u < p.nseq;
}

__device__ __forceinline__ int chunk_len(const Params& p, int c)
{
    const int64_t c0 = static_cast<int64_t>(c) * p.Q;
    return static_cast<int>(p.Q < p.T - c0 ? p.Q : p.T - c0);
}

// Per chunk and head: x4 = coefficient applied to the state at the chunk end,
// y = unit (sequence id, or batch row) of the chunk's last token,
// z = 1 when the last segment starts a sequence (reset), w = 1 when the
// chunk's last token is the last token of its unit.
// dt of token index `idx` of head h, after the block path's parameterisation
// (bias, softplus, clamp) when one is requested.
template <typename T>
__device__ __forceinline__ float load_dt(const Params& p, int64_t idx, int h)
{
    float v = Act<T>::load(static_cast<const T*>(p.dt), idx);
    if (p.dtx.active) {
        if (p.dtx.bias) v += p.dtx.bias[h];
        if (p.dtx.softplus) v = softplus_f(v);
        v = fminf(fmaxf(v, p.dtx.lo), p.dtx.hi);
    }
    return v;
}

template <typename T>
__global__ __launch_bounds__(kThreads) void k_chunk_prep(Params p)
{
    const int c = blockIdx.x, h = blockIdx.y, b = blockIdx.z, t = threadIdx.x;
    const int64_t c0 = static_cast<int64_t>(c) * p.Q;
    const int L = chunk_len(p, c);
    // this path has no bounded waits: its status is always fine
    if (p.status && c == 0 && h == 0 && b == 0 && t == 0) *p.status = 0;
    __shared__ float scr[kThreads / 64];
    __shared__ float cs_s[kThreads];
    __shared__ int q_s[kThreads];
    __shared__ int k0_s;

    const float A2 = -expf(p.A_log[h]) * kLog2e;
    float a2 = 0.f;
    if (t < L)
        a2 = load_dt<T>(p, (b * p.T + c0 + t) * p.H + h, h) * A2;
    const float cs = block_inclusive_scan(a2, scr);
    if (t < p.Q) p.cs[((b * p.H + h) * p.nC + c) * p.Q + t] = cs;
    cs_s[t] = cs;
    q_s[t] = (p.seq_idx && t < L) ? p.seq_idx[c0 + t] : 0;
    if (t == 0) k0_s = 0;
    __syncthreads();
    if (p.seq_idx && t > 0 && t < L && q_s[t] != q_s[t - 1]) atomicMax(&k0_s, t);
    __syncthreads();
    if (t == 0) {
        const int k0 = k0_s;
        int unit = b;
        int reset = 0;
        int ends = (c0 + L == p.T);
        if (p.seq_idx) {
            unit = q_s[L - 1];
            reset = (k0 > 0) || (c > 0 && p.seq_idx[c0 - 1] != q_s[0]);
            ends = ends || (p.seq_idx[c0 + L] != unit);
        }
        const float base = (reset && k0 > 0) ? cs_s[k0 - 1] : 0.f;
        const float coef = exp2f(cs_s[L - 1] - base);
        p.info[(b * p.H + h) * p.nC + c] = make_int4(__float_as_int(coef), unit, reset, ends);
    }
}

// G[t][s] = sum_n C_t[n] B_s[n] for 16x16 tiles with s-tile <= t-tile; one
// workgroup per 16-token strip of t, its s-tiles dealt to the wavefronts.  The
// operands come straight from global memory as 16-byte pieces of rows: lane
// group g takes columns 16 k + 4 g .. + 3, one per matrix instruction (the same
// permutation of the contraction on both sides).  Bound by those loads'
// latency (the whole Gram is a few per cent of the forward's products), hence
// a workgroup per strip: at 2 x 2048 tokens, N 128, float32 13 us, where one
// workgroup per chunk with 4-byte loads took 236.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_gram(Params p, int split)
{
    const int nq = static_cast<int>(p.Q / 16);
    const int c = blockIdx.x / split, g = blockIdx.y, b = blockIdx.z;
    const int lane = threadIdx.x & 63, r = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t c0 = static_cast<int64_t>(c) * p.Q;
    const int L = chunk_len(p, c), N = static_cast<int>(p.N);
    const int64_t row = p.G * p.N;
    const T* Bp = static_cast<const T*>(p.B) + ((b * p.T + c0) * p.G + g) * p.N + 4 * lg;
    const T* Cp = static_cast<const T*>(p.C) + ((b * p.T + c0) * p.G + g) * p.N + 4 * lg;
    float* Gp = p.gram + ((b * p.G + g) * p.nC + c) * p.Q * p.Q;
    // (strips past a partial chunk: tiles that no token reads)
    for (int i = blockIdx.x % split; i < nq && 16 * i < L; i += split) {
        const int t = 16 * i + r;
        const T* crow = Cp + (t < L ? t : L - 1) * row;
        for (int j = wave; j <= i; j += kThreads / 64) {
            const int s = 16 * j + r;
            const T* brow = Bp + (s < L ? s : L - 1) * row;
            f32x4_t acc = zero4();
#pragma unroll 4
            for (int k = 0; k < N; k += 16) {
                const f32x4_t cv = load4(crow + k), bv = load4(brow + k);
#pragma unroll
                for (int v = 0; v < 4; ++v) acc = mma4(bv[v], cv[v], acc);
            }
            settle(acc);
            // lane: row t, columns 16 j + 4 lg .. + 3 (rows past a partial chunk: zeros)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (t >= L || 16 * j + 4 * lg + v >= L) acc[v] = 0.f;
            store4(Gp + t * p.Q + 16 * j + 4 * lg, acc);
        }
    }
}

// Right factors run on 64 x 64 tiles (features x columns) of the P x N state,
// one workgroup each, a 2 x 2 block of 16 x 16 tiles per wavefront.  The
// tokens arrive in slabs of 64, x scaled by its weight, both token-major in
// LDS with a row stride of 80 floats (the four rows that one matrix
// instruction's operand reads fall in different banks).  Bound by the float32
// matrix rate: at 2 x 2048 tokens, 24 heads, P 64, N 128 26 us for 1.6 GFLOP;
// the 4-byte loads and one workgroup per whole state that it replaces took 142.
constexpr int kTile = 64;
constexpr int kTS = kTile + 16;

struct StateSmem {
    float X[kSlab * kTS], B[kSlab * kTS];
};

__host__ __device__ __forceinline__ int state_tiles(int64_t P, int64_t N)
{
    return static_cast<int>(((P + kTile - 1) / kTile) * ((N + kTile - 1) / kTile));
}

// Sum over the tokens s of [st, en] of w_s x_s B_s^T over tile `tile` of the
// (P x N) state, w_s = dt_s exp2(cs2_en - cs2_s); the result (plus hin_scale *
// hin, when hin is given) is stored to dst (P x N, row-major).  Block-uniform call.
template <typename T>
__device__ void segment_state(const Params& p, int b, int c, int h, int g, int tile, int st, int en,
                              const float* cs_s, const float* dt_s, float* w_s, StateSmem& sm, float* dst,
                              const float* hin, float hin_scale)
{
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int P = static_cast<int>(p.P), N = static_cast<int>(p.N);
    const int ntn = (N + kTile - 1) / kTile;
    const int p0 = (tile / ntn) * kTile, n0 = (tile % ntn) * kTile;
    const int64_t c0 = static_cast<int64_t>(c) * p.Q;
    const T* xp = static_cast<const T*>(p.x) + ((b * p.T + c0) * p.H + h) * p.P + p0;
    const T* Bp = static_cast<const T*>(p.B) + ((b * p.T + c0) * p.G + g) * p.N + n0;
    const int64_t xrow = p.H * p.P, brow = p.G * p.N;
    const int pw = 32 * (wave & 1), nw = 32 * (wave >> 1);   // this wavefront's 32 x 32 of the tile

    for (int t = tid; t < kMaxQ; t += kThreads)
        w_s[t] = (t >= st && t <= en) ? dt_s[t] * exp2f(cs_s[en] - cs_s[t]) : 0.f;
    __syncthreads();

    f32x4_t acc[2][2];   // [p-tile][n-tile]: lane holds S[p = r][n = 4 lg + v]
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = zero4();

    for (int s0 = (st / kSlab) * kSlab; s0 <= en; s0 += kSlab) {
        constexpr int kPer = kSlab * kTile / 4 / kThreads;   // 4-wide pieces per thread
        f32x4_t vx[kPer], vb[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = tid + kThreads * k, s = s0 + i / (kTile / 4), f = 4 * (i % (kTile / 4));
            vx[k] = vb[k] = zero4();
            if (s >= st && s <= en) {
                if (p0 + f < P) vx[k] = load4(xp + s * xrow + f);
                if (n0 + f < N) vb[k] = load4(Bp + s * brow + f);
            }
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = tid + kThreads * k, ss = i / (kTile / 4), f = 4 * (i % (kTile / 4));
            const float ws = w_s[s0 + ss];
            *reinterpret_cast<f32x4_t*>(&sm.X[ss * kTS + f]) = f32x4_t{vx[k][0] * ws, vx[k][1] * ws, vx[k][2] * ws, vx[k][3] * ws};
            *reinterpret_cast<f32x4_t*>(&sm.B[ss * kTS + f]) = vb[k];
        }
        __syncthreads();
#pragma unroll 4
        for (int k = 0; k < kSlab / 4; ++k) {
            const float* xr = &sm.X[(4 * k + lg) * kTS + pw + r];
            const float* br = &sm.B[(4 * k + lg) * kTS + nw + r];
            const float x0 = xr[0], x1 = xr[16], b0 = br[0], b1 = br[16];
            acc[0][0] = mma4(b0, x0, acc[0][0]);
            acc[0][1] = mma4(b1, x0, acc[0][1]);
            acc[1][0] = mma4(b0, x1, acc[1][0]);
            acc[1][1] = mma4(b1, x1, acc[1][1]);
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            settle(acc[i][j]);
            const int pp = p0 + pw + 16 * i + r, n = n0 + nw + 16 * j + 4 * lg;
            if (pp < P && n < N) {
                f32x4_t val = acc[i][j];
                if (hin) {
                    const f32x4_t hv = load4(hin + pp * N + n);
#pragma unroll
                    for (int v = 0; v < 4; ++v) val[v] += hin_scale * hv[v];
                }
                store4(dst + pp * N + n, val);
            }
        }
    __syncthreads();
}

// Shared-memory staging of one chunk's per-token scalars.
struct ChunkScalars {
    float cs[kMaxQ], dt[kMaxQ], w[kMaxQ];
    int q[kMaxQ];
};

template <typename T>
__device__ __forceinline__ void load_chunk_scalars(const Params& p, int b, int c, int h, int L,
                                                   ChunkScalars& sh)
{
    const int t = threadIdx.x;
    const int64_t c0 = static_cast<int64_t>(c) * p.Q;
    if (t < L) {
        sh.cs[t] = p.cs[((b * p.H + h) * p.nC + c) * p.Q + t];
        sh.dt[t] = load_dt<T>(p, (b * p.T + c0 + t) * p.H + h, h);
        sh.q[t] = p.seq_idx ? p.seq_idx[c0 + t] : 0;
    }
    __syncthreads();
}

// Right factors: the chunk's state at its last token from a zero start,
// restricted to the chunk's last segment.  blockIdx.x: chunk and state tile.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_chunk_state(Params p, int split)
{
    const int tiles = state_tiles(p.P, p.N);
    const int c = blockIdx.x / split, h = blockIdx.y, b = blockIdx.z;
    const int g = static_cast<int>(h / (p.H / p.G));
    const int L = chunk_len(p, c);
    __shared__ ChunkScalars sh;
    __shared__ __attribute__((aligned(16))) StateSmem sm;
    load_chunk_scalars<T>(p, b, c, h, L, sh);
    int st = 0;
    if (p.seq_idx)
        for (int k = L - 1; k > 0; --k)
            if (sh.q[k - 1] != sh.q[k]) { st = k; break; }
    float* dst = p.states + ((b * p.nC + c) * p.H + h) * p.P * p.N;
    for (int tile = blockIdx.x % split; tile < tiles; tile += split)
        segment_state<T>(p, b, c, h, g, tile, st, L - 1, sh.cs, sh.dt, sh.w, sm, dst, nullptr, 0.f);
}

// Packed rows: final states of sequences that end before their chunk's last
// token (those ending on a chunk's last token come out of the scan).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_varlen_final(Params p, int split)
{
    const int tiles = state_tiles(p.P, p.N);
    const int c = blockIdx.x / split, h = blockIdx.y, b = blockIdx.z;
    const int g = static_cast<int>(h / (p.H / p.G));
    const int64_t c0 = static_cast<int64_t>(c) * p.Q;
    const int L = chunk_len(p, c);
    const int64_t PN = p.P * p.N;
    __shared__ ChunkScalars sh;
    __shared__ __attribute__((aligned(16))) StateSmem sm;
    load_chunk_scalars<T>(p, b, c, h, L, sh);
    int st = 0;
    for (int en = 0; en < L - 1; ++en) {
        if (sh.q[en] == sh.q[en + 1]) continue;
        const int q = sh.q[en];
        const bool cont = (st == 0) && (c == 0 || p.seq_idx[c0 - 1] == q);
        const float* hin = cont ? p.states + ((b * p.nC + c) * p.H + h) * PN
                                : (p.init && unit_ok(p, q) ? p.init + (static_cast<int64_t>(q) * p.H + h) * PN : nullptr);
        const float base = (st > 0) ? sh.cs[st - 1] : 0.f;
        if (!unit_ok(p, q)) { st = en + 1; continue; }
        for (int tile = blockIdx.x % split; tile < tiles; tile += split)
            segment_state<T>(p, b, c, h, g, tile, st, en, sh.cs, sh.dt, sh.w, sm,
                             p.fin + (static_cast<int64_t>(q) * p.H + h) * PN, hin,
                             exp2f(sh.cs[en] - base));
        st = en + 1;
    }
}

// h_{-1} = initial state of the row (or of the first sequence); per chunk:
// store the entering state over the chunk state, then h = coef h + S (or
// coef * init[unit] + S after a reset); write final states at unit ends.
__global__ __launch_bounds__(kThreads) void k_state_scan(Params p)
{
    const int64_t PN = p.P * p.N;
    const int64_t idx = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    const int h = blockIdx.y, b = blockIdx.z;
    if (idx >= PN) return;
    float hs = 0.f;
    if (p.init) {
        const int64_t u0 = p.seq_idx ? p.seq_idx[0] : b;
        if (unit_ok(p, u0)) hs = p.init[(u0 * p.H + h) * PN + idx];
    }
    // the chunk terms of kAhead chunks are requested together: the walk is a
    // chain of one multiply-add a chunk, bound by the loads' latency otherwise
    constexpr int kAhead = 8;
    for (int64_t cb = 0; cb < p.nC; cb += kAhead) {
        float S[kAhead];
        int4 inf[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int64_t c = cb + k < p.nC ? cb + k : p.nC - 1;
            S[k] = p.states[((b * p.nC + c) * p.H + h) * PN + idx];
            inf[k] = p.info[(b * p.H + h) * p.nC + c];
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            if (cb + k >= p.nC) break;
            p.states[((b * p.nC + cb + k) * p.H + h) * PN + idx] = hs;
            const float coef = __int_as_float(inf[k].x);
            const bool uok = unit_ok(p, inf[k].y);
            if (inf[k].z)
                hs = (p.init && uok ? coef * p.init[(static_cast<int64_t>(inf[k].y) * p.H + h) * PN + idx] : 0.f) + S[k];
            else
                hs = coef * hs + S[k];
            if (inf[k].w && p.fin && uok) p.fin[(static_cast<int64_t>(inf[k].y) * p.H + h) * PN + idx] = hs;
        }
    }
}

// Diagonal block, left factor, skip term and store of four 16-token strips of
// a chunk, one per wavefront, for one head.  The strips of a workgroup are
// {z, 2m-1-z, 2m+z, 4m-1-z} of the chunk's 4m (equal causal work for every z),
// dealt to the wavefronts in an order that turns with the head, so that the
// longest strips do not all fall on one SIMD.  Everything is computed
// transposed, Y^T[p][t] (lane: token 16 i + r, features 16 pt + 4 lg .. + 3),
// so that a Gram row piece of four consecutive s, as loaded, is the operand of
// four matrix instructions after its mask (contraction slot of lane group lg in
// instruction v: s = 4 lg + v), with x^T read from the slab of 64 tokens in LDS
// (row stride P + 4 floats: the four rows of an operand in different banks).
// The entering state is staged in column blocks of 64.  Bound by the float32
// matrix rate: at 2 x 2048 tokens, 24 heads, P 64, N 128, Q 256 75 us for 3.3
// GFLOP, where one workgroup per chunk with 4-byte loads took 418.
template <typename T, int PT>
__global__ __launch_bounds__(kThreads) void k_chunk_output(Params p, int split)
{
    constexpr int P = 16 * PT, XS = P + 4, HS = kNB + 4;
    const int nq = static_cast<int>(p.Q / 16), nz = nq >= 4 ? nq / 4 : 1;
    const int c = blockIdx.x / split, h = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
    const int lane = tid & 63, r = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = static_cast<int>(h / (p.H / p.G));
    const int64_t c0 = static_cast<int64_t>(c) * p.Q;
    const int L = chunk_len(p, c), N = static_cast<int>(p.N);
    const int64_t PN = p.P * p.N, xrow = p.H * P, crow = p.G * p.N;
    const T* xp = static_cast<const T*>(p.x) + ((b * p.T + c0) * p.H + h) * P;
    const T* Cp = static_cast<const T*>(p.C) + ((b * p.T + c0) * p.G + g) * p.N;
    const float* Gp = p.gram + ((b * p.G + g) * p.nC + c) * p.Q * p.Q;
    __shared__ __attribute__((aligned(16))) float cs_s[kMaxQ], dt_s[kMaxQ];
    __shared__ __attribute__((aligned(16))) int q_s[kMaxQ];
    __shared__ __attribute__((aligned(16))) float xs[kSlab * XS];
    __shared__ __attribute__((aligned(16))) float hs[P * HS];

    {
        const bool in = tid < L;
        cs_s[tid] = in ? p.cs[((b * p.H + h) * p.nC + c) * p.Q + tid] : 0.f;
        dt_s[tid] = in ? load_dt<T>(p, (b * p.T + c0 + tid) * p.H + h, h) : 0.f;
        q_s[tid] = (p.seq_idx && in) ? p.seq_idx[c0 + tid] : 0;
    }
    for (int z = blockIdx.x % split; z < nz; z += split) {
        const int turn = (wave + h + c) & 3;
        const int i = turn == 0 ? z : turn == 1 ? 2 * nz - 1 - z : turn == 2 ? 2 * nz + z : 4 * nz - 1 - z;
        const int t = 16 * i + r;
        const bool mine = i < nq && 16 * i < L;          // (uniform) this wavefront has a strip
        const int last = 16 * (4 * nz - 1 - z) + 15;     // the workgroup's last token
        const int send = last < L ? last + 1 : L;
        __syncthreads();   // the chunk's scalars are in place (and the previous strips' reads done)
        const float cst = t < kMaxQ ? cs_s[t] : 0.f;
        const int qt = t < kMaxQ ? q_s[t] : 0;

        f32x4_t y[PT];
#pragma unroll
        for (int pt = 0; pt < PT; ++pt) y[pt] = zero4();

        // diagonal block: Y^T[p][t] = sum_s x^T[p][s] * (G[t][s] L_ts dt_s)
        for (int s0 = 0; s0 < send; s0 += kSlab) {
            constexpr int kPieces = kSlab * P / 4, kPer = (kPieces + kThreads - 1) / kThreads;
            f32x4_t vx[kPer];
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int e = tid + kThreads * k, s = s0 + e / (P / 4), f = 4 * (e % (P / 4));
                vx[k] = zero4();
                if (e < kPieces && s < L) vx[k] = load4(xp + s * xrow + f);
            }
            if (s0 > 0) __syncthreads();   // the previous slab's reads are done
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int e = tid + kThreads * k;
                if (e < kPieces) *reinterpret_cast<f32x4_t*>(&xs[(e / (P / 4)) * XS + 4 * (e % (P / 4))]) = vx[k];
            }
            __syncthreads();
            if (mine) {
                const float* grow = Gp + t * p.Q + s0 + 4 * lg;
                const int nj = min(kSlab / 16, i - s0 / 16 + 1);   // (may be <= 0: the strip ends before the slab)
                for (int j = 0; j < nj; ++j) {
                    const f32x4_t gv = *reinterpret_cast<const f32x4_t*>(grow + 16 * j);
                    const int s = s0 + 16 * j + 4 * lg;
                    const f32x4_t csv = *reinterpret_cast<const f32x4_t*>(&cs_s[s]);
                    const f32x4_t dtv = *reinterpret_cast<const f32x4_t*>(&dt_s[s]);
                    float m[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const bool on = s + v <= t && t < L && (!p.seq_idx || q_s[s + v] == qt);
                        m[v] = on ? gv[v] * exp2f(cst - csv[v]) * dtv[v] : 0.f;
                    }
                    const float* xr = &xs[(16 * j + 4 * lg) * XS + r];
#pragma unroll
                    for (int v = 0; v < 4; ++v)
#pragma unroll
                        for (int pt = 0; pt < PT; ++pt) y[pt] = mma4(xr[v * XS + 16 * pt], m[v], y[pt]);
                }
            }
        }

        // left factors: per segment, Y^T[p][t] += scale_t * sum_n hin[p][n] C_t[n]
        const T* ct = Cp + static_cast<int64_t>(t < L ? t : L - 1) * crow + 4 * lg;
        int st = 0;
        while (st < send) {
            int en = L - 1;
            if (p.seq_idx) {
                en = st;
                while (en + 1 < L && q_s[en + 1] == q_s[st]) ++en;
            }
            const int q = q_s[st];
            const bool cont = (st == 0) && (c == 0 || !p.seq_idx || p.seq_idx[c0 - 1] == q);
            const float* hin = cont ? p.states + ((b * p.nC + c) * p.H + h) * PN
                                    : (p.init && unit_ok(p, q) ? p.init + (static_cast<int64_t>(q) * p.H + h) * PN : nullptr);
            const float base = (st > 0) ? cs_s[st - 1] : 0.f;
            if (hin) {
                const bool reach = mine && 16 * i + 15 >= st && 16 * i <= en;
                f32x4_t tmp[PT];
#pragma unroll
                for (int pt = 0; pt < PT; ++pt) tmp[pt] = zero4();
                for (int n0 = 0; n0 < N; n0 += kNB) {
                    constexpr int kPieces = P * kNB / 4, kPer = kPieces / kThreads;
                    static_assert(kPer * kThreads == kPieces, "even split");
                    f32x4_t vh[kPer];
#pragma unroll
                    for (int k = 0; k < kPer; ++k) {
                        const int e = tid + kThreads * k, f = 4 * (e % (kNB / 4));
                        vh[k] = zero4();
                        if (n0 + f < N) vh[k] = load4(hin + (e / (kNB / 4)) * N + n0 + f);
                    }
                    __syncthreads();   // the previous block's reads are done
#pragma unroll
                    for (int k = 0; k < kPer; ++k) {
                        const int e = tid + kThreads * k;
                        *reinterpret_cast<f32x4_t*>(&hs[(e / (kNB / 4)) * HS + 4 * (e % (kNB / 4))]) = vh[k];
                    }
                    __syncthreads();
                    if (reach) {
                        const int nk = min(kNB, N - n0) / 16;
                        for (int k = 0; k < nk; ++k) {
                            const f32x4_t cv = load4(ct + n0 + 16 * k);
#pragma unroll
                            for (int pt = 0; pt < PT; ++pt) {
                                const f32x4_t hv =
                                    *reinterpret_cast<const f32x4_t*>(&hs[(16 * pt + r) * HS + 16 * k + 4 * lg]);
#pragma unroll
                                for (int v = 0; v < 4; ++v) tmp[pt] = mma4(hv[v], cv[v], tmp[pt]);
                            }
                        }
                    }
                }
                const float scale = (t >= st && t <= en) ? exp2f(cst - base) : 0.f;
#pragma unroll
                for (int pt = 0; pt < PT; ++pt) {
                    settle(tmp[pt]);
                    settle(y[pt]);
#pragma unroll
                    for (int v = 0; v < 4; ++v) y[pt][v] += scale * tmp[pt][v];
                }
            }
            st = en + 1;
        }

        // skip term and store
        if (mine && t < L) {
            const float Dh = p.D ? p.D[h] : 0.f;
            T* yp = static_cast<T*>(p.y) + ((b * p.T + c0 + t) * p.H + h) * P + 4 * lg;
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) {
                const f32x4_t xv = load4(xp + t * xrow + 16 * pt + 4 * lg);
                settle(y[pt]);
#pragma unroll
                for (int v = 0; v < 4; ++v) y[pt][v] += Dh * xv[v];
                store4(yp + 16 * pt, y[pt]);
            }
        }
    }
}

template <typename T>
hipError_t launch_all(const Params& p, hipStream_t stream, hipEvent_t ev_begin, hipEvent_t ev_end)
{
    const dim3 blk(kThreads);
    const unsigned H = static_cast<unsigned>(p.H), nb = static_cast<unsigned>(p.b);
    const dim3 g_chunk(static_cast<unsigned>(p.nC), H, nb);
    // workgroups per chunk (one when that many chunks already fill the grid's range)
    const auto split = [&](int64_t parts) { return static_cast<int>(p.nC * parts <= (1 << 23) ? parts : 1); };
    const int nq = static_cast<int>(p.Q / 16);
    const int sp_gram = split(nq), sp_state = split(state_tiles(p.P, p.N)), sp_out = split(nq >= 4 ? nq / 4 : 1);
    const dim3 g_gram(static_cast<unsigned>(p.nC * sp_gram), static_cast<unsigned>(p.G), nb);
    const dim3 g_state(static_cast<unsigned>(p.nC * sp_state), H, nb);
    const dim3 g_out(static_cast<unsigned>(p.nC * sp_out), H, nb);
    const dim3 g_scan(static_cast<unsigned>((p.P * p.N + kThreads - 1) / kThreads),
                      static_cast<unsigned>(p.H), static_cast<unsigned>(p.b));
    hipLaunchKernelGGL(k_chunk_prep<T>, g_chunk, blk, 0, stream, p);
    hipLaunchKernelGGL(k_gram<T>, g_gram, blk, 0, stream, p, sp_gram);
    hipLaunchKernelGGL(k_chunk_state<T>, g_state, blk, 0, stream, p, sp_state);
    hipLaunchKernelGGL(k_state_scan, g_scan, blk, 0, stream, p);
    hipError_t err = hipGetLastError();
    if (err == hipSuccess && ev_begin) err = hipEventRecord(ev_begin, stream);
    if (err != hipSuccess) return err;
    switch (p.P / 16) {
    case 1: hipLaunchKernelGGL((k_chunk_output<T, 1>), g_out, blk, 0, stream, p, sp_out); break;
    case 2: hipLaunchKernelGGL((k_chunk_output<T, 2>), g_out, blk, 0, stream, p, sp_out); break;
    case 3: hipLaunchKernelGGL((k_chunk_output<T, 3>), g_out, blk, 0, stream, p, sp_out); break;
    case 4: hipLaunchKernelGGL((k_chunk_output<T, 4>), g_out, blk, 0, stream, p, sp_out); break;
    case 5: hipLaunchKernelGGL((k_chunk_output<T, 5>), g_out, blk, 0, stream, p, sp_out); break;
    case 6: hipLaunchKernelGGL((k_chunk_output<T, 6>), g_out, blk, 0, stream, p, sp_out); break;
    case 7: hipLaunchKernelGGL((k_chunk_output<T, 7>), g_out, blk, 0, stream, p, sp_out); break;
    default: hipLaunchKernelGGL((k_chunk_output<T, 8>), g_out, blk, 0, stream, p, sp_out); break;
    }
    err = hipGetLastError();
    if (err == hipSuccess && ev_end) err = hipEventRecord(ev_end, stream);
    if (err != hipSuccess) return err;
    if (p.seq_idx && p.fin) hipLaunchKernelGGL(k_varlen_final<T>, g_state, blk, 0, stream, p, sp_state);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_unfused(const Params& p, bool bf16, hipStream_t stream, hipEvent_t ev_begin,
                          hipEvent_t ev_end)
{
    return bf16 ? launch_all<uint16_t>(p, stream, ev_begin, ev_end)
                : launch_all<float>(p, stream, ev_begin, ev_end);
}

}  // namespace ssd

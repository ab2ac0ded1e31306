// Gradients of the SSD layer, in the chunked form of the adjoint of its
// recurrence.  The paper gives the layer's training cost (Section 6.3) but no
// backward algorithm; this is the reverse-mode derivative of the chunked block
// decomposition of Section 6, chunk by chunk.
//
// Per (batch row, head), with chunks of Q = kBwdQ tokens, a_t = dt_t A,
// cs_t = chunk-local inclusive sum of a, e(u,t) = exp(cs_u - cs_t) (u >= t),
// X~_t = dt_t x_t, h_in the state entering the chunk, h_out the state leaving
// it and Gn the gradient of the loss with respect to h_out:
//
//   states      H_c = sum_s e(end,s) X~_s B_s^T           (h_out = exp(cs_end) h_in + H_c)
//               W_c = sum_u exp(cs_u) dy_u C_u^T          (what the chunk's outputs add to
//                                                          the gradient of h_in)
//   scans       h_in(c+1) = exp(cs_end(c)) h_in(c) + H_c,     from the initial state
//               Gn(c-1)   = exp(cs_end(c)) Gn(c) + W_c,       from the final-state gradient;
//               the gradient of the initial state is exp(cs_end(0)) Gn(0) + W_0
//   chunk       with G0(u,t) = C_u . B_t, R0(u,t) = dy_u . X~_t,
//               Gs = e G0, Rs = e R0, l(u,t) = e G0 R0 (all for u >= t):
//     dX~_t = sum_u Gs(u,t) dy_u + e(end,t) Gn B_t,       dx_t = dt_t dX~_t + D dy_t
//     dB_t  = sum_u Rs(u,t) C_u  + e(end,t) Gn^T X~_t     (summed over a group's heads)
//     dC_u  = sum_t Rs(u,t) B_t  + exp(cs_u) h_in^T dy_u  (summed over a group's heads)
//     dcs_t = sum_s l(t,s) - sum_u l(u,t) + exp(cs_t) dy_t . (h_in C_t)
//             - e(end,t) X~_t . (Gn B_t) + [t = end] <Gn, h_out>,
//     <Gn, h_out> = exp(cs_end) <Gn, h_in> + sum_s e(end,s) X~_s . (Gn B_s),
//     da_k = sum_{t >= k} dcs_t,  ddt_k = x_k . dX~_k + A da_k,
//     dA = sum dt_k da_k,  dA_log = A dA,  dD = sum dy . x.
//
// Kernels (chunks of 64 tokens, every contraction on the float32 matrix
// instructions, operands in float32 whatever the activation dtype):
//   k_bwd_gram    G0 of every chunk and group, transposed (t, u)
//   k_bwd_states  H_c and W_c, per 64 x 64 tile of the state
//   k_bwd_scan    both scans
//   k_bwd_bc      dB and dC of 64 state columns, a workgroup walking a slice of
//                 a group's heads; also dy_u . (h_in C_u) and <Gn, h_in> over
//                 its columns
//   k_bwd_dx      dx, ddt and the per-chunk terms of dA and dD, per head
//   k_bwd_reduce_bc, k_bwd_reduce_head  sums over slices, chunks and rows in a
//                 fixed order: results are deterministic.
// One float32 matrix instruction contracts four indices; here contraction slot
// of lane group q in instruction v of a 16-wide step is index 4 q + v, so that
// an operand whose rows hold the contraction index contiguously comes as one
// 16-byte read for four instructions, and a result tile (lane group q holds
// rows 4 q .. 4 q + 3) is the operand of the next product as it is.  64-wide
// rows in shared memory are 68 floats apart: 16-byte reads of 16 rows, and
// 4-byte reads of rows 4 q + v, both fall in different banks.
// A diagonal score tile (u-tile = t-tile) holds pairs with u < t, whose scores are
// zero.  Zero times an infinity is NaN, so where an operand of the chunk is not
// finite, the products over that tile run pair by pair on the vector unit.
#include "ssd_bwd.h"
#include "ssd_device.h"

namespace ssd {
namespace {

constexpr int kQ = static_cast<int>(kBwdQ);
constexpr int kThreads = 256;
constexpr int kBcThreads = 512;
constexpr int kTile = 64;            // state tile: features x columns
constexpr int kTS = kTile + 16;      // row stride of the state kernel's operands (rows 4 k + q)
constexpr int kLd = kTile + 4;       // row stride of 64-wide rows elsewhere

template <typename T>
__device__ __forceinline__ float ld(const void* p, int64_t i) { return Act<T>::load(static_cast<const T*>(p), i); }

template <typename T>
__device__ __forceinline__ void st(void* p, int64_t i, float v) { Act<T>::store(static_cast<T*>(p), i, v); }

__device__ __forceinline__ int chunk_len(int64_t T, int64_t c)
{
    const int64_t r = T - c * kQ;
    return static_cast<int>(r < kQ ? r : kQ);
}

// Sum over the 256 threads of the block in a fixed order.
__device__ __forceinline__ float block_sum256(float v, float* scr)
{
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) scr[threadIdx.x >> 6] = v;
    __syncthreads();
    const float s = (scr[0] + scr[1]) + (scr[2] + scr[3]);
    __syncthreads();
    return s;
}

// Zero if v is finite, else NaN; added up over a thread's values and over the
// wavefront: whether all of them are.
__device__ __forceinline__ float unless_finite(f32x4_t v)
{
    return fmaf(v[0], 0.f, fmaf(v[1], 0.f, fmaf(v[2], 0.f, v[3] * 0.f)));
}

__device__ __forceinline__ int any_not_finite(float z) { return __any(z != 0.f); }

// Double through DPP and readlane, half by half.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp64(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(u), CTRL, ROWS, 0xF, false);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(u >> 32), CTRL, ROWS, 0xF, false);
    return __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32 | lo);
}

__device__ __forceinline__ double lane_value64(double v, int lane)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<int>(u), lane);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<int>(u >> 32), lane);
    return __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32 | lo);
}

// A chunk's dt and inclusive cumsum of dt A (log2 units), lane = token.  The
// cumsum is kept in 64 bits and rounded only as a difference: in 32 bits its
// rounding, some 4e-6 at the end of a chunk of 64 tokens, went into every
// decay (dA_log 2e-6 off, against 1e-6 with chunks of 32).
struct TokenScan {
    float dt;
    double cs, csend;
};

template <typename T>
__device__ __forceinline__ TokenScan token_scan(const BwdParams& p, int64_t t0, int64_t h, int L, int lane)
{
    TokenScan s;
    s.dt = lane < L ? ld<T>(p.dt, (t0 + lane) * p.H + h) : 0.f;
    double v = static_cast<double>(s.dt) * static_cast<double>(-expf(p.A_log[h]) * kLog2e);
    // (the prefix sum of wave_scan)
    v += dpp64<0x111, 0xF>(v);
    v += dpp64<0x112, 0xF>(v);
    v += dpp64<0x114, 0xF>(v);
    v += dpp64<0x118, 0xF>(v);
    v += dpp64<0x142, 0xA>(v);
    v += dpp64<0x143, 0xC>(v);
    s.cs = v;
    s.csend = lane_value64(v, L - 1);
    return s;
}

__device__ __forceinline__ float decay_of(double e) { return exp2f(static_cast<float>(e)); }

// G0^T of a chunk and group: row t, columns u (u-tile >= t-tile), float32.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_bwd_gram(BwdParams p)
{
    const int64_t c = blockIdx.x, b = blockIdx.y, g = blockIdx.z;
    const int lane = threadIdx.x & 63, r = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int L = chunk_len(p.T, c), N = static_cast<int>(p.N);
    const int64_t t0 = b * p.T + c * kQ, row = p.G * p.N;
    const T* Bp = static_cast<const T*>(p.B) + (t0 * p.G + g) * p.N + 4 * q;
    const T* Cp = static_cast<const T*>(p.C) + (t0 * p.G + g) * p.N + 4 * q;
    float* out = p.gram + ((b * p.G + g) * p.nC + c) * kQ * kQ;
    const int t = 16 * w + r;
    if (16 * w >= L) return;
    const T* brow = Bp + (t < L ? t : L - 1) * row;
    for (int uj = w; 16 * uj < L && uj < kQ / 16; ++uj) {
        const int u = 16 * uj + r;
        const T* crow = Cp + (u < L ? u : L - 1) * row;
        f32x4_t acc = zero4();
#pragma unroll 4
        for (int k = 0; k < N; k += 16) {
            const f32x4_t cv = load4(crow + k), bv = load4(brow + k);
#pragma unroll
            for (int v = 0; v < 4; ++v) acc = mma4(cv[v], bv[v], acc);
        }
        settle(acc);
        store4(out + t * kQ + 16 * uj + 4 * q, acc);   // (pairs past the chunk's end are never used)
    }
}

__host__ __device__ __forceinline__ int tiles64(int64_t n) { return static_cast<int>((n + kTile - 1) / kTile); }

// Per (chunk, batch row, head, state tile, direction): H_c (into hin) or W_c
// (into gn), and the chunk's decay.  A 64 x 64 tile of the state per workgroup,
// a 2 x 2 block of 16 x 16 tiles per wavefront; weighted x (or dy) and B (or C)
// token-major in shared memory.  Bound by the float32 matrix rate and the
// states written: at 2 x 2048 tokens, 24 heads, P 64, N 128, float32 both
// directions 55 us, where one thread per state element took 254.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_bwd_states(BwdParams p, int split)
{
    __shared__ __attribute__((aligned(16))) float X[kQ * kTS];
    __shared__ __attribute__((aligned(16))) float Y[kQ * kTS];
    __shared__ float wt[kQ];
    const int ntn = tiles64(p.N), parts = 2 * tiles64(p.P) * ntn;
    const int64_t c = blockIdx.x / split, b = blockIdx.y, h = blockIdx.z, g = h / (p.H / p.G);
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = chunk_len(p.T, c), P = static_cast<int>(p.P), N = static_cast<int>(p.N);
    const int64_t t0 = b * p.T + c * kQ, bh = b * p.H + h;
    const int64_t xrow = p.H * p.P, yrow = p.G * p.N;
    const int pw = 32 * (w & 1), nw = 32 * (w >> 1);
    for (int part = blockIdx.x % split; part < parts; part += split) {
        const int dir = part & 1, p0 = ((part >> 1) / ntn) * kTile, n0 = ((part >> 1) % ntn) * kTile;
        const T* xp = static_cast<const T*>(dir == 0 ? p.x : p.dy) + (t0 * p.H + h) * p.P + p0;
        const T* yp = static_cast<const T*>(dir == 0 ? p.B : p.C) + (t0 * p.G + g) * p.N + n0;
        constexpr int kPer = kQ * kTile / 4 / kThreads;
        f32x4_t vx[kPer], vy[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = tid + kThreads * k, s = i / (kTile / 4), f = 4 * (i % (kTile / 4));
            vx[k] = vy[k] = zero4();
            if (s < L) {
                if (p0 + f < P) vx[k] = load4(xp + s * xrow + f);
                if (n0 + f < N) vy[k] = load4(yp + s * yrow + f);
            }
        }
        if (w == 0) {
            const TokenScan sc = token_scan<T>(p, t0, h, L, lane);
            wt[lane] = dir == 0 ? decay_of(sc.csend - sc.cs) * sc.dt : decay_of(sc.cs);
            if (part == 0 && lane == 0) p.cs[bh * p.nC + c] = decay_of(sc.csend);
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int i = tid + kThreads * k, s = i / (kTile / 4), f = 4 * (i % (kTile / 4));
            const float ws = wt[s];
            *reinterpret_cast<f32x4_t*>(&X[s * kTS + f]) = f32x4_t{vx[k][0] * ws, vx[k][1] * ws, vx[k][2] * ws, vx[k][3] * ws};
            *reinterpret_cast<f32x4_t*>(&Y[s * kTS + f]) = vy[k];
        }
        __syncthreads();
        f32x4_t acc[2][2];   // [p-tile][n-tile]: lane holds S[p = r][n = 4 q + v]
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = zero4();
#pragma unroll
        for (int k = 0; k < kQ / 4; ++k) {
            const float* xr = &X[(4 * k + q) * kTS + pw + r];
            const float* yr = &Y[(4 * k + q) * kTS + nw + r];
            const float x0 = xr[0], x1 = xr[16], y0 = yr[0], y1 = yr[16];
            acc[0][0] = mma4(y0, x0, acc[0][0]);
            acc[0][1] = mma4(y1, x0, acc[0][1]);
            acc[1][0] = mma4(y0, x1, acc[1][0]);
            acc[1][1] = mma4(y1, x1, acc[1][1]);
        }
        float* dst = (dir == 0 ? p.hin : p.gn) + ((b * p.nC + c) * p.H + h) * p.P * p.N;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int pp = p0 + pw + 16 * i + r, n = n0 + nw + 16 * j + 4 * q;
                if (pp < P && n < N) store4(dst + pp * N + n, acc[i][j]);
            }
        if (split < parts) __syncthreads();   // (uniform) before the next part overwrites the operands
    }
}

// The scans over chunks, one thread per 4 consecutive state elements of one
// (batch row, head) and direction, in place: hin(c) <- state entering chunk c,
// gn(c) <- gradient of the state leaving chunk c; direction 1 writes dinit.
// The terms of kAhead chunks are requested together (a chain of one
// multiply-add a chunk, bound by the loads otherwise).
__global__ __launch_bounds__(kThreads) void k_bwd_scan(BwdParams p)
{
    constexpr int kAhead = 4;
    const int64_t PN4 = p.P * p.N / 4;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (i >= p.b * p.H * PN4) return;
    const int dir = blockIdx.y;
    const int64_t bh = i / PN4, e4 = i - bh * PN4;
    const int64_t b = bh / p.H, h = bh - b * p.H;
    const int64_t stride = p.H * PN4;       // between consecutive chunks, in float4
    float4* a = reinterpret_cast<float4*>(dir == 0 ? p.hin : p.gn) + (b * p.nC * p.H + h) * PN4 + e4;
    const float* dec = p.cs + bh * p.nC;
    const float* start = dir == 0 ? p.init : p.dfinal;
    float4 acc = start ? reinterpret_cast<const float4*>(start)[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    const auto at = [&](int64_t k) { return dir == 0 ? k : p.nC - 1 - k; };
    for (int64_t k0 = 0; k0 < p.nC; k0 += kAhead) {
        float4 loc[kAhead];
        float d[kAhead];
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            const int64_t c = at(k0 + k < p.nC ? k0 + k : p.nC - 1);
            loc[k] = a[c * stride];
            d[k] = dec[c];
        }
#pragma unroll
        for (int k = 0; k < kAhead; ++k) {
            if (k0 + k >= p.nC) break;
            a[at(k0 + k) * stride] = acc;
            acc.x = fmaf(d[k], acc.x, loc[k].x);
            acc.y = fmaf(d[k], acc.y, loc[k].y);
            acc.z = fmaf(d[k], acc.z, loc[k].z);
            acc.w = fmaf(d[k], acc.w, loc[k].w);
        }
    }
    if (dir == 1 && p.dinit) reinterpret_cast<float4*>(p.dinit)[i] = acc;
}

// The score tiles (u-tile, t-tile) with u >= t: wavefront w takes tile w and,
// for w < 2, tile w + 8.
__constant__ int2 kScoreTile[10] = {{0, 0}, {1, 0}, {1, 1}, {2, 0}, {2, 1}, {2, 2}, {3, 0}, {3, 1}, {3, 2}, {3, 3}};

// dB and dC of 64 state columns of a chunk, summed over a slice of a group's
// heads in registers (wavefront w: n-tile w / 2, tokens of tiles 2 (w % 2) and
// 2 (w % 2) + 1).  Per head: R0 = dy x^T, Gn^T x^T and h_in^T dy^T over the head's
// features in blocks of 64, then Rs = e R0 dt through shared memory into C^T Rs
// and B^T Rs^T.  The next block of x, dy, Gn and h_in is fetched while this one
// is multiplied.  Bound by the float32 matrix rate (about 300 instructions of
// 32 cycles per SIMD and head): at 2 x 2048 tokens, 24 heads, P 64, N 128 106
// us; the kernel of float32 FMAs on shared memory that this and k_bwd_dx
// replace took 3069.
template <typename T>
__global__ __launch_bounds__(kBcThreads) void k_bwd_bc(BwdParams p, int split)
{
    __shared__ __attribute__((aligned(16))) float xs[kQ * kLd];    // x   (row t, features)
    __shared__ __attribute__((aligned(16))) float dys[kQ * kLd];   // dy  (row u, features)
    __shared__ __attribute__((aligned(16))) float Gs[kTile * kLd]; // Gn  (row feature, columns)
    __shared__ __attribute__((aligned(16))) float Hs[kTile * kLd]; // h_in
    __shared__ __attribute__((aligned(16))) float Bs[kQ * kLd];    // B   (row t, columns)
    __shared__ __attribute__((aligned(16))) float Cs[kQ * kLd];    // C
    __shared__ __attribute__((aligned(16))) float Rs[kQ * kLd];    // Rs  (row u, columns t <= u)
    __shared__ double scs[kQ];
    __shared__ float sdt[kQ], seend[kQ], secs[kQ], q1s[kQ][4], scr[8];
    __shared__ int sbad[2][8];           // B, C not finite, by wavefront
    const int nb_all = tiles64(p.N);
    const int64_t c = blockIdx.x / split, b = blockIdx.y;
    const int64_t hpg = p.H / p.G, g = blockIdx.z / p.S, slice = blockIdx.z - g * p.S;
    const int64_t h_lo = g * hpg + slice * p.hs;
    const int64_t h_hi = (slice + 1) * p.hs < hpg ? h_lo + p.hs : g * hpg + hpg;
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, q = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = chunk_len(p.T, c), P = static_cast<int>(p.P), N = static_cast<int>(p.N);
    const int64_t t0 = b * p.T + c * kQ, xrow = p.H * p.P, yrow = p.G * p.N;
    const int nt = w >> 1, tp = 2 * (w & 1);
    const int ntile = w < 2 ? 2 : 1;
    constexpr int kPer = kQ * kTile / 4 / kBcThreads;   // 2 pieces of 4 per thread and array
    const int row0 = tid / (kTile / 4), col = 4 * (tid % (kTile / 4));   // piece k: row row0 + 32 k

    for (int nb = blockIdx.x % split; nb < nb_all; nb += split) {
        const int n0 = nb * kTile;
        const bool cols = n0 + 16 * nt < N;   // (uniform) this wavefront's n-tile exists
        const T* Bp = static_cast<const T*>(p.B) + (t0 * p.G + g) * p.N + n0 + col;
        const T* Cp = static_cast<const T*>(p.C) + (t0 * p.G + g) * p.N + n0 + col;
        __syncthreads();   // (a second column block: the first one's reads are done)
        float zb = 0.f, zc = 0.f;
        int bad_b = 0, bad_c = 0;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int s = row0 + 32 * k;
            f32x4_t vb = zero4(), vc = zero4();
            if (s < L && n0 + col < N) {
                vb = load4(Bp + s * yrow);
                vc = load4(Cp + s * yrow);
            }
            *reinterpret_cast<f32x4_t*>(&Bs[s * kLd + col]) = vb;
            *reinterpret_cast<f32x4_t*>(&Cs[s * kLd + col]) = vc;
            zb += unless_finite(vb);
            zc += unless_finite(vc);
        }
        const int nzb = any_not_finite(zb), nzc = any_not_finite(zc);
        if (lane == 0) {
            sbad[0][w] = nzb;
            sbad[1][w] = nzc;
        }
        f32x4_t dB[2], dC[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) dB[j] = dC[j] = zero4();

        // features p0 .. p0 + 63 of head h
        f32x4_t fx[kPer], fd[kPer], fg[kPer], fh[kPer];
        const auto fetch = [&](int64_t h, int p0) {
            const T* xp = static_cast<const T*>(p.x) + (t0 * p.H + h) * p.P + p0 + col;
            const T* dp = static_cast<const T*>(p.dy) + (t0 * p.H + h) * p.P + p0 + col;
            const int64_t sb = ((b * p.nC + c) * p.H + h) * p.P * p.N + static_cast<int64_t>(p0) * N + n0 + col;
#pragma unroll
            for (int k = 0; k < kPer; ++k) {
                const int s = row0 + 32 * k;
                fx[k] = fd[k] = fg[k] = fh[k] = zero4();
                if (s < L && p0 + col < P) {
                    fx[k] = load4(xp + s * xrow);
                    fd[k] = load4(dp + s * xrow);
                }
                if (p0 + s < P && n0 + col < N) {
                    fg[k] = load4(p.gn + sb + s * N);
                    fh[k] = load4(p.hin + sb + s * N);
                }
            }
        };
        fetch(h_lo, 0);
        for (int64_t h = h_lo; h < h_hi; ++h) {
            if (w == 0) {   // (every wavefront is past the previous head's last barrier)
                const TokenScan sc = token_scan<T>(p, t0, h, L, lane);
                scs[lane] = sc.cs;
                sdt[lane] = sc.dt;
                seend[lane] = lane < L ? decay_of(sc.csend - sc.cs) : 0.f;
                secs[lane] = lane < L ? decay_of(sc.cs) : 0.f;
            }
            f32x4_t r0[2], bx[2], ch[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) r0[j] = bx[j] = ch[j] = zero4();
            float gh = 0.f;
            for (int p0 = 0; p0 < P; p0 += kTile) {
                if (p0 > 0) __syncthreads();   // the previous block's reads are done
#pragma unroll
                for (int k = 0; k < kPer; ++k) {
                    const int s = row0 + 32 * k;
                    *reinterpret_cast<f32x4_t*>(&xs[s * kLd + col]) = fx[k];
                    *reinterpret_cast<f32x4_t*>(&dys[s * kLd + col]) = fd[k];
                    *reinterpret_cast<f32x4_t*>(&Gs[s * kLd + col]) = fg[k];
                    *reinterpret_cast<f32x4_t*>(&Hs[s * kLd + col]) = fh[k];
#pragma unroll
                    for (int v = 0; v < 4; ++v) gh = fmaf(fg[k][v], fh[k][v], gh);
                }
                if (p0 + kTile < P)
                    fetch(h, p0 + kTile);
                else if (h + 1 < h_hi)
                    fetch(h + 1, 0);
                __syncthreads();
                const int kp = min(kTile, P - p0) / 16;
                // (rolled: unrolled, the operand reads of all steps are hoisted and spill)
#pragma unroll 1
                for (int k = 0; k < kp; ++k) {
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        if (j < ntile) {
                            const int2 tl = kScoreTile[w + 8 * j];
                            const f32x4_t dv = *reinterpret_cast<const f32x4_t*>(&dys[(16 * tl.x + r) * kLd + 16 * k + 4 * q]);
                            const f32x4_t xv = *reinterpret_cast<const f32x4_t*>(&xs[(16 * tl.y + r) * kLd + 16 * k + 4 * q]);
#pragma unroll
                            for (int v = 0; v < 4; ++v) r0[j] = mma4(dv[v], xv[v], r0[j]);
                        }
                    if (cols) {
                        f32x4_t xv[2], dv[2];
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            xv[j] = *reinterpret_cast<const f32x4_t*>(&xs[(16 * (tp + j) + r) * kLd + 16 * k + 4 * q]);
                            dv[j] = *reinterpret_cast<const f32x4_t*>(&dys[(16 * (tp + j) + r) * kLd + 16 * k + 4 * q]);
                        }
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const float gv = Gs[(16 * k + 4 * q + v) * kLd + 16 * nt + r];
                            const float hv = Hs[(16 * k + 4 * q + v) * kLd + 16 * nt + r];
#pragma unroll
                            for (int j = 0; j < 2; ++j) {
                                bx[j] = mma4(gv, xv[j][v], bx[j]);
                                ch[j] = mma4(hv, dv[j][v], ch[j]);
                            }
                        }
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                settle(r0[j]);
                settle(bx[j]);
                settle(ch[j]);
            }
            // Rs = e(u, t) R0 dt_t on u >= t
#pragma unroll
            for (int j = 0; j < 2; ++j)
                if (j < ntile) {
                    const int2 tl = kScoreTile[w + 8 * j];
                    const int t = 16 * tl.y + r;
                    const float dtt = sdt[t];
                    const double cst = scs[t];
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int u = 16 * tl.x + 4 * q + v;
                        Rs[u * kLd + t] = u >= t && u < L ? decay_of(scs[u] - cst) * (r0[j][v] * dtt) : 0.f;
                    }
                }
            gh = wave_sum(gh);
            if (lane == 0) scr[w] = gh;
            if (h == h_lo) {   // (stored before the barriers of this head's blocks)
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    bad_b |= sbad[0][k];
                    bad_c |= sbad[1][k];
                }
                bad_b = __builtin_amdgcn_readfirstlane(bad_b);
                bad_c = __builtin_amdgcn_readfirstlane(bad_c);
            }
            __syncthreads();
            if (cols) {
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int tt = tp + j, t = 16 * tt + r;
                    // dB^T(n, t) += sum over u >= t of C^T Rs
#pragma unroll 1
                    for (int uj = tt + bad_c; uj < kQ / 16; ++uj)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int u = 16 * uj + 4 * q + v;
                            dB[j] = mma4(Cs[u * kLd + 16 * nt + r], Rs[u * kLd + t], dB[j]);
                        }
                    // dC^T(n, u = t) += sum over s <= u of B^T Rs^T
#pragma unroll 1
                    for (int sj = 0; sj + bad_b <= tt; ++sj) {
                        const f32x4_t rv = *reinterpret_cast<const f32x4_t*>(&Rs[t * kLd + 16 * sj + 4 * q]);
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            dC[j] = mma4(Bs[(16 * sj + 4 * q + v) * kLd + 16 * nt + r], rv[v], dC[j]);
                    }
                    const f32x4_t cv = *reinterpret_cast<const f32x4_t*>(&Cs[t * kLd + 16 * nt + 4 * q]);
                    const float fb = seend[t] * sdt[t], fc = secs[t];
                    float q1 = 0.f;
                    settle(dB[j]);
                    settle(dC[j]);
                    if (bad_c) {   // the diagonal tile, pair by pair
#pragma unroll 1
                        for (int u = 16 * tt; u < 16 * tt + 16; ++u)
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                if (u >= t) dB[j][v] = fmaf(Cs[u * kLd + 16 * nt + 4 * q + v], Rs[u * kLd + t], dB[j][v]);
                    }
                    if (bad_b) {
#pragma unroll 1
                        for (int s1 = 16 * tt; s1 < 16 * tt + 16; ++s1)
#pragma unroll
                            for (int v = 0; v < 4; ++v)
                                if (s1 <= t) dC[j][v] = fmaf(Bs[s1 * kLd + 16 * nt + 4 * q + v], Rs[t * kLd + s1], dC[j][v]);
                    }
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        dB[j][v] = fmaf(fb, bx[j][v], dB[j][v]);
                        dC[j][v] = fmaf(fc, ch[j][v], dC[j][v]);
                        q1 = fmaf(cv[v], ch[j][v], q1);
                    }
                    q1 = col_sum4(q1);   // dy_u . (h_in C_u) over this n-tile
                    if (q == 0) q1s[t][nt] = q1;
                }
            } else if (q == 0) {
                q1s[16 * tp + r][nt] = 0.f;
                q1s[16 * (tp + 1) + r][nt] = 0.f;
            }
            __syncthreads();
            const int64_t slot = (static_cast<int64_t>(nb) * p.b + b) * p.H + h;
            if (w == 1 && lane < L)
                p.q1p[slot * p.T + c * kQ + lane] = (q1s[lane][0] + q1s[lane][1]) + (q1s[lane][2] + q1s[lane][3]);
            if (tid == 128) p.ghp[slot * p.nC + c] = ((scr[0] + scr[1]) + (scr[2] + scr[3])) + ((scr[4] + scr[5]) + (scr[6] + scr[7]));
        }
        // this slice's dB and dC: lane holds n = n0 + 16 nt + 4 q .. + 3, token 16 tt + r;
        // with one slice per group they are the gradients
        if (cols)
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int t = 16 * (tp + j) + r;
                if (t < L) {
                    const int64_t o = ((t0 + t) * p.G + g) * p.N + n0 + 16 * nt + 4 * q;
                    if (p.S == 1) {
                        store4(static_cast<T*>(p.dB) + o, dB[j]);
                        store4(static_cast<T*>(p.dC) + o, dC[j]);
                    } else {
                        const int64_t so = slice * p.b * p.T * p.G * p.N + o;
                        store4(p.dBp + so, dB[j]);
                        store4(p.dCp + so, dC[j]);
                    }
                }
            }
    }
}

// dx, ddt and the chunk's terms of dA and dD for one head (after k_bwd_bc).
// Wavefronts own the t-tiles, in an order that turns with the head (a tile's
// work falls with t); everything is transposed (lane: token t, features
// 16 pt + 4 q .. + 3), so that a score tile Gs, as computed, is the operand of
// dy^T Gs.  Gn is staged in column blocks of 64.  Bound by the float32 matrix
// rate: at 2 x 2048 tokens, 24 heads, P 64, N 128 61 us.
template <typename T, int PT>
__global__ __launch_bounds__(kThreads) void k_bwd_dx(BwdParams p)
{
    constexpr int P = 16 * PT, XS = P + 4;
    __shared__ __attribute__((aligned(16))) float xs[kQ * XS];
    __shared__ __attribute__((aligned(16))) float dys[kQ * XS];
    __shared__ __attribute__((aligned(16))) float Gs[P * kLd];
    __shared__ double scs[kQ];
    __shared__ float sdt[kQ], seend[kQ], secs[kQ], xdx[kQ], q2s[kQ], dyxs[kQ], cols[kQ], rowp[kQ][4], scr[4];
    __shared__ int sbad[4];              // dy not finite, by wavefront
    const int64_t c = blockIdx.x, b = blockIdx.y, h = blockIdx.z, g = h / (p.H / p.G), bh = b * p.H + h;
    const int tid = threadIdx.x, lane = tid & 63, r = lane & 15, q = lane >> 4;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = (wv + static_cast<int>(h + c)) & 3;   // this wavefront's t-tile
    const int L = chunk_len(p.T, c), N = static_cast<int>(p.N);
    const int64_t t0 = b * p.T + c * kQ, xrow = p.H * P;
    const T* xp = static_cast<const T*>(p.x) + (t0 * p.H + h) * P;
    const T* dp = static_cast<const T*>(p.dy) + (t0 * p.H + h) * P;
    const int t = 16 * w + r;

    constexpr int kPer = kQ * P / 4 / kThreads;
    {
        f32x4_t vx[kPer], vd[kPer];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int e = tid + kThreads * k, s = e / (P / 4), f = 4 * (e % (P / 4));
            vx[k] = vd[k] = zero4();
            if (s < L) {
                vx[k] = load4(xp + s * xrow + f);
                vd[k] = load4(dp + s * xrow + f);
            }
        }
        if (wv == 0) {
            const TokenScan sc = token_scan<T>(p, t0, h, L, lane);
            scs[lane] = sc.cs;
            sdt[lane] = sc.dt;
            seend[lane] = lane < L ? decay_of(sc.csend - sc.cs) : 0.f;
            secs[lane] = lane < L ? decay_of(sc.cs) : 0.f;
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int e = tid + kThreads * k, s = e / (P / 4), f = 4 * (e % (P / 4));
            *reinterpret_cast<f32x4_t*>(&xs[s * XS + f]) = vx[k];
            *reinterpret_cast<f32x4_t*>(&dys[s * XS + f]) = vd[k];
        }
        float z = 0.f;
#pragma unroll
        for (int k = 0; k < kPer; ++k) z += unless_finite(vd[k]);
        const int nz = any_not_finite(z);
        if (lane == 0) sbad[wv] = nz;
    }
    __syncthreads();
    const int bad = __builtin_amdgcn_readfirstlane(sbad[0] | sbad[1] | sbad[2] | sbad[3]);

    // scores on the tiles u >= t of this t-tile: Gs into dy^T Gs, l into its row and column sums
    f32x4_t ai[PT], ag[PT];
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) ai[pt] = ag[pt] = zero4();
    const float* grow = p.gram + (((b * p.G + g) * p.nC + c) * kQ + t) * kQ + 4 * q;
    const float dtt = sdt[t];
    const double cst = scs[t];
    float colsum = 0.f, asum = 0.f;
#pragma unroll
    for (int uj = 0; uj < kQ / 16; ++uj) {
        if (uj < w || 16 * uj >= L) continue;   // (uniform)
        const f32x4_t gv = *reinterpret_cast<const f32x4_t*>(grow + 16 * uj);
        f32x4_t r0 = zero4();
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const f32x4_t dv = *reinterpret_cast<const f32x4_t*>(&dys[(16 * uj + r) * XS + 16 * k + 4 * q]);
            const f32x4_t xv = *reinterpret_cast<const f32x4_t*>(&xs[t * XS + 16 * k + 4 * q]);
#pragma unroll
            for (int v = 0; v < 4; ++v) r0 = mma4(dv[v], xv[v], r0);
        }
        settle(r0);
        float gs[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int u = 16 * uj + 4 * q + v;
            float lv = 0.f;
            gs[v] = 0.f;
            if (u >= t && u < L) {
                const float ex = static_cast<float>(scs[u] - cst);
                gs[v] = exp2f(ex) * gv[v];
                // (l(t, t) is in the row and in the column sum of token t: left out of
                // both, or its rounding would stay where the two cancel)
                if (u > t) lv = gs[v] * (r0[v] * dtt);
                asum = fmaf(lv, ex, asum);
            }
            colsum += lv;
            const float rsum = row_sum16(lv);
            if (r == 0) rowp[u][w] = rsum;
        }
        if (bad && uj == w) {   // the diagonal tile (this wavefront's first), pair by pair
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll 1
                for (int k = 0; k < 4; ++k) {
                    const int u = 16 * uj + 4 * k + v;
                    const float gut = __shfl(gs[v], 16 * k + r, 64);
#pragma unroll
                    for (int pt = 0; pt < PT; ++pt)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (u >= t) ai[pt][e] = fmaf(dys[u * XS + 16 * pt + 4 * q + e], gut, ai[pt][e]);
                }
            continue;
        }
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int pt = 0; pt < PT; ++pt)
                ai[pt] = mma4(dys[(16 * uj + 4 * q + v) * XS + 16 * pt + r], gs[v], ai[pt]);
    }
    colsum = col_sum4(colsum);
    if (q == 0) cols[t] = colsum;
    asum = wave_sum(asum);
    if (lane == 0) scr[w] = asum;

    // Gn B^T
    const T* brow = static_cast<const T*>(p.B) + ((t0 + (t < L ? t : L - 1)) * p.G + g) * p.N + 4 * q;
    const float* Gn = p.gn + ((b * p.nC + c) * p.H + h) * P * p.N;
    for (int n0 = 0; n0 < N; n0 += kTile) {
        constexpr int kG = P * kTile / 4 / kThreads;
        f32x4_t vg[kG];
#pragma unroll
        for (int k = 0; k < kG; ++k) {
            const int e = tid + kThreads * k, f = 4 * (e % (kTile / 4));
            vg[k] = zero4();
            if (n0 + f < N) vg[k] = load4(Gn + (e / (kTile / 4)) * N + n0 + f);
        }
        if (n0 > 0) __syncthreads();   // the previous block's reads are done
#pragma unroll
        for (int k = 0; k < kG; ++k) {
            const int e = tid + kThreads * k;
            *reinterpret_cast<f32x4_t*>(&Gs[(e / (kTile / 4)) * kLd + 4 * (e % (kTile / 4))]) = vg[k];
        }
        __syncthreads();
        const int nk = min(kTile, N - n0) / 16;
#pragma unroll 1
        for (int k = 0; k < nk; ++k) {
            const f32x4_t bv = load4(brow + n0 + 16 * k);
#pragma unroll
            for (int pt = 0; pt < PT; ++pt) {
                const f32x4_t gv = *reinterpret_cast<const f32x4_t*>(&Gs[(16 * pt + r) * kLd + 16 * k + 4 * q]);
#pragma unroll
                for (int v = 0; v < 4; ++v) ag[pt] = mma4(gv[v], bv[v], ag[pt]);
            }
        }
    }

    // dX~ and dx; per-token sums over the features
    const float Ah = -expf(p.A_log[h]);
    const float Dh = p.D ? p.D[h] : 0.f;
    const float ee = seend[t];
    float sxd = 0.f, sxg = 0.f, sdx = 0.f;
#pragma unroll
    for (int pt = 0; pt < PT; ++pt) {
        settle(ai[pt]);
        settle(ag[pt]);
        const f32x4_t xv = *reinterpret_cast<const f32x4_t*>(&xs[t * XS + 16 * pt + 4 * q]);
        const f32x4_t dv = *reinterpret_cast<const f32x4_t*>(&dys[t * XS + 16 * pt + 4 * q]);
        f32x4_t dx;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const float dX = fmaf(ee, ag[pt][v], ai[pt][v]);
            dx[v] = fmaf(dtt, dX, Dh * dv[v]);
            sxd = fmaf(xv[v], dX, sxd);
            sxg = fmaf(xv[v], ag[pt][v], sxg);
            sdx = fmaf(dv[v], xv[v], sdx);
        }
        if (t < L) store4(static_cast<T*>(p.dx) + ((t0 + t) * p.H + h) * P + 16 * pt + 4 * q, dx);
    }
    sxd = col_sum4(sxd);
    sxg = col_sum4(sxg);
    sdx = col_sum4(sdx);
    if (q == 0) {
        xdx[t] = sxd;
        q2s[t] = sxg;
        dyxs[t] = sdx;
    }
    __syncthreads();

    // per token (lane k holds token 63 - k, so that a prefix sum over lanes is a
    // suffix sum over tokens): dcs, then the decay gradients
    if (wv == 0) {
        const int tk = kQ - 1 - lane;
        const bool in = tk < L;
        float q1 = 0.f, ghs = 0.f, row = 0.f;
        for (int nb = 0; nb < tiles64(N); ++nb) {
            const int64_t slot = (static_cast<int64_t>(nb) * p.b + b) * p.H + h;
            if (in) q1 += p.q1p[slot * p.T + c * kQ + tk];
            ghs += p.ghp[slot * p.nC + c];
        }
        const float q2 = in ? sdt[tk] * q2s[tk] : 0.f;   // X~_t . (Gn B_t)
        const float hsum = wave_sum(seend[tk] * q2);
        if (in)
            for (int k = 0; k <= tk / 16; ++k) row += rowp[tk][k];
        float dcs = in ? row - cols[tk] + secs[tk] * q1 - seend[tk] * q2 : 0.f;
        if (tk == L - 1) dcs += secs[tk] * ghs + hsum;   // <Gn, h_out>
        const float da = wave_scan(dcs);                 // over tokens t' >= t
        if (in) st<T>(p.ddt, (t0 + tk) * p.H + h, fmaf(Ah, da, xdx[tk]));
        // dA = sum of dt da, term by term: a pair (u, t) is in da of the tokens t + 1
        // .. u, whose dt add up to its exponent over A, and likewise for the
        // other terms of dcs.  (The sum of dt da itself is what little of large
        // terms cancels.)  Exponents in log2 units, hence 1 / (A log2 e); an A that
        // has underflowed to zero has no gradient through A_log.
        const float cst2 = static_cast<float>(scs[tk]), cse = static_cast<float>(scs[L - 1]);
        float at = in ? secs[tk] * q1 * cst2 + seend[tk] * q2 * static_cast<float>(scs[L - 1] - scs[tk]) : 0.f;
        if (tk == L - 1) at += secs[tk] * ghs * cse;
        const float asum4 = wave_sum(at) + ((scr[0] + scr[1]) + (scr[2] + scr[3]));
        const float sa = Ah != 0.f ? asum4 / (Ah * kLog2e) : 0.f;
        const float sd = wave_sum(in ? dyxs[tk] : 0.f);
        if (lane == 0) {
            p.dAp[bh * p.nC + c] = sa;
            p.dDp[bh * p.nC + c] = sd;
        }
    }
}

// dB, dC = sum over head slices (fixed order), rounded to the input dtype.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_bwd_reduce_bc(BwdParams p)
{
    const int64_t n_el = p.b * p.T * p.G * p.N;
    const int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (i >= n_el) return;
    float sb = 0.f, sc = 0.f;
    for (int64_t s = 0; s < p.S; ++s) {
        sb += p.dBp[s * n_el + i];
        sc += p.dCp[s * n_el + i];
    }
    st<T>(p.dB, i, sb);
    st<T>(p.dC, i, sc);
}

// dA_log[h] = A_h * sum over rows and chunks of the dA terms; dD likewise.
__global__ __launch_bounds__(kThreads) void k_bwd_reduce_head(BwdParams p)
{
    __shared__ float scr[4];
    const int64_t h = blockIdx.x;
    float sa = 0.f, sd = 0.f;
    for (int64_t i = threadIdx.x; i < p.b * p.nC; i += kThreads) {
        const int64_t b = i / p.nC, c = i - b * p.nC;
        sa += p.dAp[(b * p.H + h) * p.nC + c];
        sd += p.dDp[(b * p.H + h) * p.nC + c];
    }
    sa = block_sum256(sa, scr);
    sd = block_sum256(sd, scr);
    if (threadIdx.x == 0) {
        p.dA_log[h] = -expf(p.A_log[h]) * sa;
        if (p.dD) p.dD[h] = sd;
    }
}

template <typename T>
hipError_t launch_all(const BwdParams& p, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1)
{
    const unsigned nC = static_cast<unsigned>(p.nC), nb = static_cast<unsigned>(p.b), H = static_cast<unsigned>(p.H);
    // workgroups per chunk (one when that many chunks already fill the grid's range)
    const auto split = [&](int64_t parts) { return static_cast<int>(p.nC * parts <= (1 << 22) ? parts : 1); };
    const int sp_state = split(2 * tiles64(p.P) * tiles64(p.N)), sp_bc = split(tiles64(p.N));
    hipLaunchKernelGGL(k_bwd_gram<T>, dim3(nC, nb, static_cast<unsigned>(p.G)), dim3(kThreads), 0, st, p);
    hipLaunchKernelGGL(k_bwd_states<T>, dim3(nC * static_cast<unsigned>(sp_state), nb, H), dim3(kThreads), 0, st, p,
                       sp_state);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nscan = p.b * p.H * p.P * p.N / 4;
    hipLaunchKernelGGL(k_bwd_scan, dim3(static_cast<unsigned>((nscan + kThreads - 1) / kThreads), 2), dim3(kThreads),
                       0, st, p);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev0 && (e = hipEventRecord(ev0, st)) != hipSuccess) return e;
    hipLaunchKernelGGL(k_bwd_bc<T>, dim3(nC * static_cast<unsigned>(sp_bc), nb, static_cast<unsigned>(p.G * p.S)),
                       dim3(kBcThreads), 0, st, p, sp_bc);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev1 && (e = hipEventRecord(ev1, st)) != hipSuccess) return e;
    const dim3 g_dx(nC, nb, H);
    const auto dx = [&](auto kern) { hipLaunchKernelGGL(kern, g_dx, dim3(kThreads), 0, st, p); };
    switch (p.P / 16) {
    case 1: dx(k_bwd_dx<T, 1>); break;
    case 2: dx(k_bwd_dx<T, 2>); break;
    case 3: dx(k_bwd_dx<T, 3>); break;
    case 4: dx(k_bwd_dx<T, 4>); break;
    case 5: dx(k_bwd_dx<T, 5>); break;
    case 6: dx(k_bwd_dx<T, 6>); break;
    case 7: dx(k_bwd_dx<T, 7>); break;
    default: dx(k_bwd_dx<T, 8>); break;
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    return launch_backward_reduce(p, sizeof(T) == 2, st, p.S > 1);
}

template <typename T>
hipError_t launch_reduce(const BwdParams& p, hipStream_t st, bool with_bc)
{
    const int64_t nbc = p.b * p.T * p.G * p.N;
    if (with_bc) {
        hipLaunchKernelGGL(k_bwd_reduce_bc<T>, dim3(static_cast<unsigned>((nbc + kThreads - 1) / kThreads)),
                           dim3(kThreads), 0, st, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_bwd_reduce_head, dim3(static_cast<unsigned>(p.H)), dim3(kThreads), 0, st, p);
    return hipGetLastError();
}

size_t al(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

void bwd_slices(int64_t b, int64_t nC, int64_t G, int64_t hpg, int64_t* S, int64_t* hs)
{
    // as few slices as still give every compute unit of the chip (256 CUs) a
    // workgroup: a workgroup shares B, C and the chunk's Gram tiles over its
    // heads and accumulates dB, dC over them (measured at the 2.7B shape, bf16:
    // 80 heads per workgroup 0.610 ms, 40: 0.629, 16: 0.667, 8: 0.726)
    constexpr int64_t kCUs = 256;
    const int64_t units = b * nC * G;
    int64_t s = (kCUs + units - 1) / units;
    if (s > hpg) s = hpg;
    if (s < 1) s = 1;
    *hs = (hpg + s - 1) / s;
    *S = (hpg + *hs - 1) / *hs;
}

BwdLayout bwd_layout(int64_t b, int64_t T, int64_t H, int64_t P, int64_t N, int64_t G, int64_t nC, int64_t S,
                     bool fast)
{
    BwdLayout l{};
    size_t off = 0;
    const auto take_bytes = [&](size_t bytes) {
        const size_t o = off;
        off += al(bytes);
        return o;
    };
    const auto take = [&](size_t n) { return take_bytes(n * sizeof(float)); };
    const size_t state_bytes = static_cast<size_t>(b * nC * H * P * N) * (fast ? 2 : 4);
    l.cs = fast ? 0 : take(static_cast<size_t>(b * H * nC));
    l.hin = take_bytes(state_bytes);
    l.gn = fast ? 0 : take_bytes(state_bytes);
    l.gnT = fast ? take_bytes(state_bytes) : 0;
    if (!fast) {
        const int64_t nblk = (N + kTile - 1) / kTile;
        l.gram = take(static_cast<size_t>(b * G * nC * kBwdQ * kBwdQ));
        l.q1p = take(static_cast<size_t>(nblk * b * H * T));
        l.ghp = take(static_cast<size_t>(nblk * b * H * nC));
    }
    l.dBp = take(static_cast<size_t>(S * b * T * G * N));
    l.dCp = take(static_cast<size_t>(S * b * T * G * N));
    l.dAp = take(static_cast<size_t>(b * nC * H));
    l.dDp = take(static_cast<size_t>(b * nC * H));
    l.total = off;
    return l;
}

namespace {

// out[c] = sum over rows r (in order) of part[r][c].
__global__ __launch_bounds__(kThreads) void k_sum_rows(const float* part, int64_t nrows, int64_t ncols, float* out)
{
    const int64_t c = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (c >= ncols) return;
    float s = 0.f;
    for (int64_t r = 0; r < nrows; ++r) s += part[r * ncols + c];
    out[c] = s;
}

}  // namespace

hipError_t launch_sum_rows(const float* part, int64_t nrows, int64_t ncols, float* out, hipStream_t stream)
{
    hipLaunchKernelGGL(k_sum_rows, dim3(static_cast<unsigned>((ncols + kThreads - 1) / kThreads)), dim3(kThreads), 0,
                       stream, part, nrows, ncols, out);
    return hipGetLastError();
}

hipError_t launch_backward_reduce(const BwdParams& p, bool bf16, hipStream_t stream, bool with_bc)
{
    return bf16 ? launch_reduce<uint16_t>(p, stream, with_bc) : launch_reduce<float>(p, stream, with_bc);
}

hipError_t launch_backward(const BwdParams& p, bool bf16, hipStream_t stream, hipEvent_t ev_begin,
                           hipEvent_t ev_end)
{
    return bf16 ? launch_all<uint16_t>(p, stream, ev_begin, ev_end)
                : launch_all<float>(p, stream, ev_begin, ev_end);
}

}  // namespace ssd

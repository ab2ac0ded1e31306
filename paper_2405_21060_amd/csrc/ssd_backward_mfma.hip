// Gradients of the SSD layer on the matrix cores: bf16 inputs, headdim 64,
// dstate 64 or 128.  Same chunked adjoint as ssd_backward.hip (formulas at the
// top of that file), with chunks of 64 tokens and every contraction on
// v_mfma_f32_16x16x32_bf16 (bf16 operands, float32 accumulation):
//
//   k_bwd2_pass    the chunk states: per (row, head, direction) a walk
//                  over the chunks with a float32 running
//                  state, writing h_in^T (forward) or Gn^T (backward, from the
//                  final-state gradient) per chunk in bf16; the initial-state
//                  gradient in float32
//   k_bwd2_chunk   per (chunk, row, group, head slice): all chunk terms.  Score
//                  tiles (u >= t) R0 = dy x^T and G0 = C B^T (once per
//                  workgroup), then dX~^T = dy^T Gs + Gn B^T, dB^T = C^T Rs +
//                  Gn^T x~^T, dC^T = B^T Rs^T + h_in^T dy^T, each as 16 x 16
//                  tiles.  B, Gn^T, x, dy and the scores lie in shared memory
//                  once, as they come, and are read by rows or transposed
//                  (ds_read_b64_tr_b16); what every head takes of C^T and B^T is
//                  in registers, h_in^T comes straight from global memory.
//
// H32 (a template flag; the block gradients use it): dt and dy come in as
// float32 and ddt goes out as float32.  dy is rounded to bf16 only where it is
// a matrix-core operand; the skip term of dx and the dD sums take it in float32.
//
// An MFMA operand row holds the contraction index contiguously; a lane
// (row r = lane % 16, group q = lane / 16) reads 8 of them (k = 32 s + 8 q ..
// + 7) as one 16-byte load, and the result tile D[4 q + v][r] lands in its
// four accumulator registers.  A transposing read gives slots 0..3 k = 32 s +
// 4 q .. + 3 and slots 4..7 k = 32 s + 16 + 4 q .. + 3 ("slot order"): the other
// operand of such a product is stored in that order.
#include <type_traits>

#include "ssd_bwd.h"
#include "ssd_device.h"

namespace ssd {
namespace {

constexpr int kQ2 = 64;          // tokens per chunk
constexpr int kP2 = 64;          // head dimension
constexpr int kT2 = 512;         // threads per workgroup (8 wavefronts)

typedef uint16_t u16;
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16x8_t frag(uint4 v) { return __builtin_bit_cast(bf16x8_t, v); }

__device__ __forceinline__ f32x4_t mma(uint4 a, uint4 b, f32x4_t c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag(a), frag(b), c, 0, 0, 0);
}

// Two floats rounded to bf16 (nearest even, one v_cvt_pk_bf16_f32), the first in
// the low half.
__device__ __forceinline__ uint32_t pack2(float lo, float hi)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    bf16x2_t v;
    v[0] = static_cast<__bf16>(lo);
    v[1] = static_cast<__bf16>(hi);
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ uint32_t bf16_bits(float f) { return pack2(f, 0.f) & 0xFFFFu; }

// dt from its raw bits (float32, or bf16 in the low half).
template <bool H32>
__device__ __forceinline__ float dt_of_raw(uint32_t v)
{
    return H32 ? __uint_as_float(v) : __uint_as_float(v << 16);
}

__device__ __forceinline__ float lo_f(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_f(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ int chunk_len2(int64_t T, int64_t c)
{
    const int64_t r = T - c * kQ2;
    return static_cast<int>(r < kQ2 ? r : kQ2);
}

// Slice of a group's heads handled by this workgroup.
struct HeadRange {
    int64_t g, slice, lo, hi;
};

__device__ __forceinline__ HeadRange head_range(const BwdParams& p)
{
    HeadRange r;
    const int64_t hpg = p.H / p.G;
    r.g = blockIdx.z / p.S;
    r.slice = blockIdx.z - r.g * p.S;
    r.lo = r.g * hpg + r.slice * p.hs;
    r.hi = (r.slice + 1) * p.hs < hpg ? r.lo + p.hs : r.g * hpg + hpg;
    return r;
}

// ---------------------------------------------------------------------------
// State passes: one workgroup per (row, head, direction) walks the chunks in
// order with a float32 running state S (64 p x N) in registers, and writes S
// (bf16, n x p) for every chunk before adding the chunk's own term:
//   direction 0 (forward, from the initial state): h_in(c) = S, then
//     S <- exp(cs_end) S + sum_s (e(end,s) dt_s x_s) B_s^T;
//   direction 1 (backward, from the final-state gradient): Gn(c) = S, then
//     S <- exp(cs_end) S + sum_u (exp(cs_u) dy_u) C_u^T;
//   at the end of direction 1, S is the initial-state gradient (float32).
// The chunk term is a 64 x N x 64 product over the chunk's tokens on the
// matrix cores.  Both operands stay token-major in shared memory (whole
// 16-byte pieces of rows, as loaded: the global loads are coalesced), with
// each row's 8-element groups XOR-swizzled by the row index, and the
// contraction fragments come out of transposing reads (ds_read_b64_tr_b16):
// within a 16-lane group, source lane j reads row k0 + j/4, elements f0 +
// 4 (j%4) .. +3, and lane i receives element f0 + i of rows k0 .. k0 + 3.
// Lane group g takes rows 4 g .. 4 g + 3 and 16 + 4 g .. 16 + 4 g + 3 of each
// 32-token step for its eight contraction slots (the same map for both
// operands).  Inputs are fetched two chunks ahead.  Wavefront w owns p rows
// 16 w .. 16 w + 15 of S (N / 16 tiles of 16 x 16).
constexpr int kPassT = 256;

typedef short v4i16 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) v4i16 lds_v4i16;

// Element offset of (row s, element f) in a token-major buffer of F elements
// per row, 8-element groups swizzled by (s & 7).
template <int F>
__device__ __forceinline__ int tok_off(int s, int f)
{
    return s * F + ((((f >> 3) ^ (s & 7)) << 3) | (f & 7));
}

// Contraction fragment over tokens 32 m .. 32 m + 31 of elements f0 .. f0 + 15.
template <int F>
__device__ __forceinline__ uint4 tr_frag(const u16* buf, int m, int f0, int lane)
{
    const int j = lane & 15, g = lane >> 4;
    const int row = 32 * m + 4 * g + (j >> 2), f = f0 + 4 * (j & 3);
    const uint2 lo = __builtin_bit_cast(
        uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(buf + tok_off<F>(row, f))));
    const uint2 hi = __builtin_bit_cast(
        uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(buf + tok_off<F>(row + 16, f))));
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
}

// PACKED: a packed row; workgroup (sequence, head) walks that sequence's
// chunks of the chunk table.
template <int N, bool PACKED, bool H32>
__global__ __launch_bounds__(kPassT, H32 ? 2 : 1) void k_bwd2_pass(BwdParams p)
{
    __shared__ __attribute__((aligned(16))) u16 XS[kQ2 * kP2];   // weighted x (or dy), token-major
    __shared__ __attribute__((aligned(16))) u16 YS[kQ2 * N];     // B (or C), token-major
    // the chunk's state (bf16, n x p) on its way out: rows padded to 72
    // elements so that the 16 n-rows of a wavefront's writes spread over the
    // banks; read back as whole 128-byte rows, so that the global stores cover
    // full rows (a wavefront's own fragments are 32-byte pieces of 16 rows)
    constexpr int kOBld = kP2 + 8;
    __shared__ __attribute__((aligned(16))) u16 OB[N * kOBld];

    const int64_t bh = blockIdx.x;
    const int64_t b = bh / p.H, h = bh - b * p.H, g = h / (p.H / p.G);
    const int dir = static_cast<int>(blockIdx.y);
    // wavefront index, provably uniform (per-wavefront choices stay scalar)
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    const u16* src = static_cast<const u16*>(dir == 0 ? p.x : p.dy);
    const float* dyf = static_cast<const float*>(p.dy);   // H32, dir 1
    const bool src32 = H32 && dir == 1;
    const u16* bc = static_cast<const u16*>(dir == 0 ? p.B : p.C);
    u16* out = reinterpret_cast<u16*>(dir == 0 ? p.hin : p.gnT);
    const float A2 = -expf(p.A_log[h]) * kLog2e;

    // running state: lane holds S[p = 16 w + 4 q + v][n = 16 nt + r]
    constexpr int kNT = N / 16;
    f32x4_t S[kNT];
    const float* s0 = dir == 0 ? p.init : p.dfinal;
#pragma unroll
    for (int nt = 0; nt < kNT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            S[nt][v] = s0 ? s0[(bh * kP2 + 16 * w + 4 * q + v) * N + 16 * nt + r] : 0.f;

    // The passes' loop, once per kind of source (the float32 dy of the block
    // gradients' direction 1 is known per workgroup): no branch on it inside
    // the loop, whose waits then count the loads in flight.
    const auto run = [&](auto s32tag) {
        constexpr bool S32 = decltype(s32tag)::value;
        // One chunk's inputs: dt (lane = token), and 16-byte pieces of x (or dy)
        // and of B (or C): piece i = tid + 256 k is row i / (F/8), group i % (F/8),
        // so consecutive lanes read consecutive bytes of a row.
        constexpr int kXK = kQ2 * kP2 / 8 / kPassT;   // 2
        constexpr int kYK = kQ2 * N / 8 / kPassT;     // N / 32
        struct Stage {
            uint32_t dt;   // raw bits (widened where used: a conversion waits for the loads before it)
            u32x4_t x[kXK], y[kYK];
            f32x4_t xf[H32 ? 2 * kXK : 1];   // H32, dir 1: dy in float32
        };
        int64_t first = 0, nch = p.nC;   // this row's (or sequence's) chunks
        if constexpr (PACKED) {
            first = p.seq_first[b];
            nch = p.seq_first[b + 1] - first;
        }
        const auto chunk_at = [&](int64_t k) { return first + (dir == 0 ? k : nch - 1 - k); };
        const auto fetch = [&](Stage& st, int64_t k) {
            // Branch-free: past the last chunk the last one is fetched again (never
            // used), and rows past a partial chunk read as zeros through the buffer
            // bounds, so that the compiler can count exactly which loads are still
            // in flight when a stage is used (with branches around them it waits
            // for all of them: the next stage's and the state stores included).
            const int64_t c = chunk_at(k < nch ? k : nch - 1);
            int L;
            int64_t t0;
            if constexpr (PACKED) {
                const int4 e = p.vtab[c];
                L = e.y;
                t0 = e.x;
            } else {
                L = chunk_len2(p.T, c);
                t0 = b * p.T + c * kQ2;
            }
            constexpr int kDtBytes = H32 ? 4 : 2;
            const __amdgpu_buffer_rsrc_t rdt = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char*>(static_cast<const char*>(p.dt)) + (t0 * p.H + h) * kDtBytes, 0,
                static_cast<int>(((L - 1) * p.H + 1) * kDtBytes), 0x00020000);
            const int dtoff = lane * static_cast<int>(p.H) * kDtBytes;
            if constexpr (H32)
                st.dt = __builtin_amdgcn_raw_buffer_load_b32(rdt, dtoff, 0, 0);
            else
                st.dt = __builtin_amdgcn_raw_buffer_load_b16(rdt, dtoff, 0, 0);
            const int xrow = static_cast<int>(p.H) * kP2;   // elements between tokens of x (dy)
    #pragma unroll
            for (int kk = 0; kk < kXK; ++kk) {
                const int i = tid + kPassT * kk, s = i >> 3, f = 8 * (i & 7);
                if constexpr (S32) {
                    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                        const_cast<float*>(dyf) + (t0 * p.H + h) * kP2, 0,
                        ((L - 1) * xrow + kP2) * static_cast<int>(sizeof(float)), 0x00020000);
                    const int off = (s * xrow + f) * static_cast<int>(sizeof(float));
                    st.xf[2 * kk] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, off, 0, 0));
                    st.xf[2 * kk + 1] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(rs, off + 16, 0, 0));
                } else {
                    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                        const_cast<u16*>(src) + (t0 * p.H + h) * kP2, 0,
                        ((L - 1) * xrow + kP2) * static_cast<int>(sizeof(u16)), 0x00020000);
                    st.x[kk] = __builtin_amdgcn_raw_buffer_load_b128(
                        rs, (s * xrow + f) * static_cast<int>(sizeof(u16)), 0, 0);
                }
            }
            const int yrow = static_cast<int>(p.G) * N;   // elements between tokens of B (C)
            const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<u16*>(bc) + (t0 * p.G + g) * N, 0, ((L - 1) * yrow + N) * static_cast<int>(sizeof(u16)),
                0x00020000);
    #pragma unroll
            for (int kk = 0; kk < kYK; ++kk) {
                const int i = tid + kPassT * kk, s = i / (N / 8), f = 8 * (i % (N / 8));
                st.y[kk] = __builtin_amdgcn_raw_buffer_load_b128(ry, (s * yrow + f) * static_cast<int>(sizeof(u16)), 0, 0);
            }
        };
        const auto step = [&](Stage& st, int64_t k) {
            const int64_t c = chunk_at(k);
            const int L = PACKED ? p.vtab[c].y : chunk_len2(p.T, c);
            // token weights: cumsum with lane = token, then each piece's token's weight
            const float dtv = dt_of_raw<H32>(st.dt);
            const float cs = wave_scan(dtv * A2);
            const float csend = lane_value(cs, L - 1);
            const float wt = dir == 0 ? exp2f(csend - cs) * dtv : exp2f(cs);
            __syncthreads();   // the previous chunk's product is done with XS, YS
    #pragma unroll
            for (int kk = 0; kk < kXK; ++kk) {
                const int i = tid + kPassT * kk, s = i >> 3, f = 8 * (i & 7);
                const float ws = __shfl(wt, s, 64);
                uint32_t o[4];
                if constexpr (S32) {
                    const f32x4_t a = st.xf[2 * kk], c2 = st.xf[2 * kk + 1];
                    o[0] = pack2(ws * a.x, ws * a.y);
                    o[1] = pack2(ws * a.z, ws * a.w);
                    o[2] = pack2(ws * c2.x, ws * c2.y);
                    o[3] = pack2(ws * c2.z, ws * c2.w);
                } else {
                    const uint32_t ex[4] = {st.x[kk].x, st.x[kk].y, st.x[kk].z, st.x[kk].w};
    #pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = pack2(ws * lo_f(ex[e]), ws * hi_f(ex[e]));
                }
                *reinterpret_cast<uint4*>(XS + tok_off<kP2>(s, f)) = make_uint4(o[0], o[1], o[2], o[3]);
            }
    #pragma unroll
            for (int kk = 0; kk < kYK; ++kk) {
                const int i = tid + kPassT * kk, s = i / (N / 8), f = 8 * (i % (N / 8));
                *reinterpret_cast<u32x4_t*>(YS + tok_off<N>(s, f)) = st.y[kk];
            }
            fetch(st, k + 2);

            // S before this chunk's term -> out(c), bf16 (n x p), through OB
    #pragma unroll
            for (int nt = 0; nt < kNT; ++nt)
                *reinterpret_cast<uint2*>(OB + (16 * nt + r) * kOBld + 16 * w + 4 * q) =
                    make_uint2(pack2(S[nt][0], S[nt][1]), pack2(S[nt][2], S[nt][3]));

            __syncthreads();   // this chunk's operands and its state in place
            {
                u16* o = out + ((PACKED ? c : b * p.nC + c) * p.H + h) * kP2 * N;
                constexpr int kOK = N * kP2 / 8 / kPassT;   // 16-byte pieces per thread
    #pragma unroll
                for (int kk = 0; kk < kOK; ++kk) {
                    const int i = tid + kPassT * kk, row = i >> 3, c8 = 8 * (i & 7);
                    // (streaming stores: 671 MB at the 2.7B shape, read once by the next
                    // kernel; the backward 604 -> 590 us, 405 -> 401 with the block's 201 MB)
                    __builtin_nontemporal_store(*reinterpret_cast<const u32x4_t*>(OB + row * kOBld + c8),
                                                reinterpret_cast<u32x4_t*>(o + row * kP2 + c8));
                }
            }
            const float a = exp2f(csend);
            const uint4 xf0 = tr_frag<kP2>(XS, 0, 16 * w, lane), xf1 = tr_frag<kP2>(XS, 1, 16 * w, lane);
    #pragma unroll
            for (int nt = 0; nt < kNT; ++nt) {
                f32x4_t t = zero4();
                t = mma(xf0, tr_frag<N>(YS, 0, 16 * nt, lane), t);
                t = mma(xf1, tr_frag<N>(YS, 1, 16 * nt, lane), t);
    #pragma unroll
                for (int v = 0; v < 4; ++v) S[nt][v] = fmaf(a, S[nt][v], t[v]);
            }
        };
        Stage s0st, s1st;
        fetch(s0st, 0);
        fetch(s1st, 1);
        // (pairs of steps, then an odd last one: no branch inside the loop body)
        int64_t k = 0;
        for (; k + 1 < nch; k += 2) {
            step(s0st, k);
            step(s1st, k + 1);
        }
        if (k < nch) step(s0st, k);
    };
    if (src32)
        run(std::true_type{});
    else
        run(std::false_type{});
    if (dir == 1 && p.dinit) {
#pragma unroll
        for (int nt = 0; nt < kNT; ++nt)
#pragma unroll
            for (int v = 0; v < 4; ++v) p.dinit[(bh * kP2 + 16 * w + 4 * q + v) * N + 16 * nt + r] = S[nt][v];
    }
}

// ---------------------------------------------------------------------------
// Chunk gradients.  Shared arrays are rows of 16-byte groups XOR-swizzled by the
// row (tok_off), each value once:
//   Bs  64 x N   B (row t), with n in the order of the transposing reads' slots
//                (perm_off): one 16-byte read is an operand of the products over n
//   Gn  N x 64   Gn^T (row n), as it lies in memory; read by rows for the products
//                over p and transposed for the one over n.  Holds C (64 x N) first.
//   xs, dys  64 x 64   x and dy (row = token)
//   Gs, Rs   64 x 64   the masked scores, row t, with u in the slots' order
// Bound by the latency of its phases and the issue of vector and shared-memory
// instructions (two wavefronts per SIMD), not by its bytes.  Transposed copies
// of B, C, dy, Gn and the scores written element by element for every head,
// software rounding, products over the zero half of the scores, and state loads
// issued at the head that uses them took 564 us at the 2.7B shape (4 x 4,096
// tokens, 80 heads); reading one copy transposed 467, with the states fetched a
// head ahead 403, and as a pipeline over the heads with one barrier a head
// instead of three 364 (exp2f for the decays, which keeps those below 2^-126,
// costs 6 of the whole backward's 602).  (128 registers, two workgroups per compute unit: 1,455
// us, the operands fetched ahead are spilled.)
template <int N>
constexpr size_t chunk_smem()
{
    return sizeof(u16) * (3 * static_cast<size_t>(kQ2) * N + (3 * 2 + 2 * 2) * kQ2 * kP2);
}

// Element offset of column 32 m + 16 h + 4 g (+ 0..3) of row s in a buffer whose
// columns lie in slot order: position 32 m + 8 g + 4 h.
template <int F>
__device__ __forceinline__ int perm_off(int s, int m, int h, int g)
{
    return tok_off<F>(s, 32 * m + 8 * g + 4 * h);
}

// Operand fragment of row `row`, k-step ks (eight consecutive positions).
template <int F>
__device__ __forceinline__ uint4 row_frag(const u16* buf, int row, int ks, int lane)
{
    return *reinterpret_cast<const uint4*>(buf + tok_off<F>(row, 32 * ks + 8 * (lane >> 4)));
}

// tr_frag of a buffer whose columns lie in slot order: columns 16 ft .. + 15.
template <int F>
__device__ __forceinline__ uint4 tr_frag_perm(const u16* buf, int m, int ft, int lane)
{
    const int j = lane & 15, g = lane >> 4, row = 32 * m + 4 * g + (j >> 2);
    const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                   (lds_v4i16*)(buf + perm_off<F>(row, ft >> 1, ft & 1, j & 3))));
    const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                                   (lds_v4i16*)(buf + perm_off<F>(row + 16, ft >> 1, ft & 1, j & 3))));
    return make_uint4(lo.x, lo.y, hi.x, hi.y);
}

// Four sums over the lane groups q at once: lane group q gets the sum of v_q
// over lanes r, r + 16, r + 32, r + 48.
__device__ __forceinline__ float col_sum4x4(float v0, float v1, float v2, float v3)
{
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v0), __float_as_uint(v2), false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v1), __float_as_uint(v3), false, false);
    const float s = __uint_as_float(a[0]) + __uint_as_float(a[1]), t = __uint_as_float(b[0]) + __uint_as_float(b[1]);
    const auto c = __builtin_amdgcn_permlane16_swap(__float_as_uint(s), __float_as_uint(t), false, false);
    return __uint_as_float(c[0]) + __uint_as_float(c[1]);
}

// Four sums over the 16 lanes of a row at once: lane r gets the sum of v_(r % 4).
__device__ __forceinline__ float row_sum16x4(float v0, float v1, float v2, float v3, int r)
{
    const bool o1 = r & 1, o2 = r & 2;
    const float a = (o1 ? v1 : v0) + dpp<0xB1, 0xF>(o1 ? v0 : v1);
    const float b = (o1 ? v3 : v2) + dpp<0xB1, 0xF>(o1 ? v2 : v3);
    float c = (o2 ? b : a) + dpp<0x4E, 0xF>(o2 ? a : b);
    c += dpp<0x124, 0xF>(c);
    c += dpp<0x128, 0xF>(c);
    return c;
}

// Byte offsets of a lane's accesses within the shared buffers (tile and k-step
// add constants): rows of 64 and of N elements by k-step, the transposing reads
// by tile pair (op) and of p-tile pw (ot), the lane's x and dy of a dX^T tile.
// Each phase works them out from its own opaque copy of the lane: the compiler
// would otherwise keep every sum with a tile's offset in a register of its own
// across the heads (100 registers spilled).
template <int N>
struct LaneOffs {
    int r, q, oa[2], ob[2], op[2], ot, ox;

    __device__ __forceinline__ LaneOffs(int lane, int pw)
    {
        asm volatile("" : "+v"(lane));
        r = lane & 15;
        q = lane >> 4;
        const int j4 = lane & 3, trow = 4 * q + (r >> 2);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            oa[ks] = 2 * tok_off<kP2>(r, 32 * ks + 8 * q);
            ob[ks] = 2 * tok_off<N>(r, 32 * ks + 8 * q);
            op[ks] = 2 * tok_off<kP2>(trow, 32 * ks + 8 * j4);
        }
        ot = 2 * tok_off<kP2>(trow, 16 * pw + 4 * j4);
        ox = 2 * tok_off<kP2>(r, 16 * pw + 4 * q);
    }
    static __device__ __forceinline__ const char* at(const u16* buf, int off)
    {
        return reinterpret_cast<const char*>(buf) + off;
    }
    __device__ __forceinline__ uint4 row64(const u16* buf, int tile, int ks) const
    {
        return *reinterpret_cast<const uint4*>(at(buf, 32 * kP2 * tile + oa[ks]));
    }
    __device__ __forceinline__ uint4 rowN(const u16* buf, int tile, int ks) const
    {
        return *reinterpret_cast<const uint4*>(at(buf, 32 * N * tile + 128 * (ks >> 1) + ob[ks & 1]));
    }
    __device__ __forceinline__ uint4 tr64(const u16* buf, int m, int off) const   // rows 32 m .. 32 m + 31
    {
        const char* a = at(buf, 64 * kP2 * m + off);
        const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)a));
        const uint2 hi =
            __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4i16*)(a + 32 * kP2)));
        return make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
};

// The score tiles (u-tile, t-tile) with u >= t, dealt to the wavefronts:
// wavefront w evaluates kLowerTile[w] and, for w >= 6, kLowerTile[w + 2]
// (wavefronts 0 and 1 have the per-token phases).
__constant__ int2 kLowerTile[10] = {{0, 0}, {1, 0}, {1, 1}, {2, 0}, {2, 1}, {2, 2}, {3, 0}, {3, 1}, {3, 2}, {3, 3}};

// DIRECT: one head slice per group; dB and dC stored by this kernel (bf16).
template <int N, bool PACKED, bool H32, bool DIRECT>
// A_log and D come as separate read-only arguments so that their per-head
// values are scalar loads: read through the parameter block (whose other
// pointers the kernel writes through) they were vector loads, and the wait for
// them at every head's start also waited for all the memory operations
// before them, the previous head's gradient stores included.
__global__ __launch_bounds__(kT2) void k_bwd2_chunk(BwdParams p, const float* __restrict__ A_logp,
                                                       const float* __restrict__ Dp)
{
    constexpr int kNT = N / 16;             // n-tiles
    constexpr int kBW = N / 32;             // dB / dC tiles per wavefront
    extern __shared__ __attribute__((aligned(16))) u16 sm2[];
    u16* const Bs = sm2;
    u16* const Gn2 = Bs + kQ2 * N;             // [2]
    u16* const xs3 = Gn2 + 2 * kQ2 * N;        // [3]
    u16* const dys3 = xs3 + 3 * kQ2 * kP2;     // [3]
    u16* const Gs2 = dys3 + 3 * kQ2 * kP2;     // [2]
    u16* const Rs2 = Gs2 + 2 * kQ2 * kP2;      // [2]
    // per-token factors, by head (mod 4): written two heads ahead, read last by the
    // per-token phase a head behind
    __shared__ __attribute__((aligned(16))) float scs4[4][kQ2], sdt4[4][kQ2], seend4[4][kQ2], secs4[4][kQ2];
    // partial sums of the per-token phase, by token within a slot: of the
    // scores by row and by column (by head mod 3), x . dX~ and x . (Gn B) by
    // p-tile, and dy . (h_in C) by n-tile; then <Gn, h_in> and dy . x by lane
    // group (by head mod 2)
    __shared__ float rowp3[3][4][kQ2], colp3[3][4][kQ2], xdp2[2][2][4][kQ2], q1p2[2][kNT][kQ2];
    __shared__ float ghp2[2][32], dyxp2[2][32];

    const int64_t c = blockIdx.x, b = blockIdx.y;
    const HeadRange hr = head_range(p);
    // wavefront index, provably uniform: the tile tables below are read with
    // scalar loads, never vector loads whose wait would also wait for the
    // next head's inputs in flight
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, q = lane >> 4;
    int L0 = 0;
    int64_t t00 = 0;
    if constexpr (PACKED) {   // chunk c of the table; entries past its end add nothing to dA, dD
        if (c >= *p.vcount) {
            for (int64_t hh = hr.lo + tid; hh < hr.hi; hh += kT2) {
                p.dAp[hh * p.nC + c] = 0.f;
                p.dDp[hh * p.nC + c] = 0.f;
            }
            return;
        }
        const int4 e = p.vtab[c];
        L0 = e.y;
        t00 = e.x;
    } else {
        L0 = chunk_len2(p.T, c);
        t00 = b * p.T + c * kQ2;
    }
    const int L = L0;
    const int64_t t0 = t00;

    // B and C of the chunk; cleared: the two score tiles above the diagonal that
    // the products read, and the partial sums of those that nobody writes
    for (int i = tid; i < kQ2 * N / 8; i += kT2) {
        const int s = i / (N / 8), n0 = 8 * (i % (N / 8));
        uint4 vb = make_uint4(0, 0, 0, 0), vc = vb;
        if (s < L) {
            const int64_t gi = ((t0 + s) * p.G + hr.g) * N + n0;
            vb = *reinterpret_cast<const uint4*>(static_cast<const u16*>(p.B) + gi);
            vc = *reinterpret_cast<const uint4*>(static_cast<const u16*>(p.C) + gi);
        }
        const int m = n0 >> 5, h = (n0 >> 4) & 1, g = (n0 >> 2) & 3;
        *reinterpret_cast<uint2*>(Bs + perm_off<N>(s, m, h, g)) = make_uint2(vb.x, vb.y);
        *reinterpret_cast<uint2*>(Bs + perm_off<N>(s, m, h, g + 1)) = make_uint2(vb.z, vb.w);
        *reinterpret_cast<uint4*>(Gn2 + tok_off<N>(s, n0)) = vc;
    }
    if (w < 4) {   // tiles (u 0, t 1) and (u 2, t 3) of Gs and Rs
        u16* const dst = w & 1 ? Rs2 : Gs2;
        const int ut = w & 2;
        for (int k = 0; k < 2; ++k)
            *reinterpret_cast<uint2*>(dst + kQ2 * kP2 * k + perm_off<kP2>(16 * (ut + 1) + r, ut >> 1, 0, q)) =
                make_uint2(0, 0);
    } else {
        for (int k = 0; k < 3; ++k) rowp3[k][w - 4][lane] = colp3[k][w - 4][lane] = 0.f;
    }
    __syncthreads();

    // G0 = C B^T on this wavefront's score tiles
    const int ntile = w >= 6 ? 2 : 1;
    f32x4_t g0[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        g0[k] = zero4();
        if (k < ntile) {
            const int2 tl = kLowerTile[w + 2 * k];
#pragma unroll
            for (int ks = 0; ks < N / 32; ++ks) {
                const uint2 lo = *reinterpret_cast<const uint2*>(Gn2 + tok_off<N>(16 * tl.x + r, 32 * ks + 4 * q));
                const uint2 hi = *reinterpret_cast<const uint2*>(Gn2 + tok_off<N>(16 * tl.x + r, 32 * ks + 16 + 4 * q));
                g0[k] = mma(make_uint4(lo.x, lo.y, hi.x, hi.y), row_frag<N>(Bs, 16 * tl.y + r, ks, lane), g0[k]);
            }
        }
    }
    const int pw = w & 3;   // p-tile of dX^T
    // What every head's dB^T and dC^T products take of B and C, in registers: this
    // wavefront's n-tile of C^T and B^T, and C where the lane's dC^T tiles lie.
    // Tile j of the wavefront is n-tile nt, token tile tile_of(j).
    const int nt = (w * kBW) >> 2;
    const auto tile_of = [&](int j) { return kBW == 4 ? j : (w & 1) + 2 * j; };
    uint4 ctf[2], btf[2];
    uint2 cv[kBW];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
        ctf[ks] = tr_frag<N>(Gn2, ks, 16 * nt, lane);
        btf[ks] = tr_frag_perm<N>(Bs, ks, nt, lane);
    }
#pragma unroll
    for (int j = 0; j < kBW; ++j)
        cv[j] = *reinterpret_cast<const uint2*>(Gn2 + tok_off<N>(16 * tile_of(j) + r, 16 * nt + 4 * q));

    f32x4_t dBacc[kBW], dCacc[kBW];
#pragma unroll
    for (int j = 0; j < kBW; ++j) dBacc[j] = dCacc[j] = zero4();

    // one head's inputs, fetched a head ahead: dt (wavefront 0, lane = token) and
    // a 16-byte piece of x and of dy per thread; rows past a partial chunk read as
    // zeros through the buffer bounds
    constexpr int kDtBytes = H32 ? 4 : 2, kDyBytes = H32 ? 4 : 2;
    const int xrow = static_cast<int>(p.H) * kP2;   // elements between tokens of x and dy
    uint32_t pdt = 0;   // raw bits, widened where used
    uint4 px = make_uint4(0, 0, 0, 0), pd = px;
    float4 pf0 = make_float4(0.f, 0.f, 0.f, 0.f), pf1 = pf0;   // H32: dy in float32
    const auto fetch = [&](int64_t h) {
        if (w == 0) {
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<char*>(static_cast<const char*>(p.dt)) + (t0 * p.H + h) * kDtBytes, 0,
                static_cast<int>(((L - 1) * p.H + 1) * kDtBytes), 0x00020000);
            const int off = lane * static_cast<int>(p.H) * kDtBytes;
            if constexpr (H32)
                pdt = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
            else
                pdt = __builtin_amdgcn_raw_buffer_load_b16(rs, off, 0, 0);
        }
        const int64_t base = (t0 * p.H + h) * kP2;
        const int off = (tid >> 3) * xrow + 8 * (tid & 7), last = (L - 1) * xrow + kP2;
        const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<u16*>(static_cast<const u16*>(p.x)) + base, 0, last * static_cast<int>(sizeof(u16)), 0x00020000);
        const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<char*>(static_cast<const char*>(p.dy)) + base * kDyBytes, 0, last * kDyBytes, 0x00020000);
        px = __builtin_bit_cast(
            uint4, __builtin_amdgcn_raw_buffer_load_b128(rx, off * static_cast<int>(sizeof(u16)), 0, 0));
        if constexpr (H32) {
            pf0 = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rd, off * kDyBytes, 0, 0));
            pf1 = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(rd, off * kDyBytes + 16, 0, 0));
        } else {
            pd = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rd, off * kDyBytes, 0, 0));
        }
    };
    const int staged = tok_off<kP2>(tid >> 3, 8 * (tid & 7));   // a thread's piece of a 64-wide buffer
    // and Gn^T (pieces for the shared copy) and this wavefront's fragments of
    // h_in^T, each fetched for the next head once this head's have been used
    u32x4_t gpc[N / 64];
    uint4 hinf[2];
    const auto state_at = [&](int64_t h) { return ((b * p.nC + c) * p.H + h) * kP2 * N; };
    const auto fetch_gn = [&](int64_t h) {
        const u16* g = reinterpret_cast<const u16*>(p.gnT) + state_at(h);
#pragma unroll
        for (int k = 0; k < N / 64; ++k) gpc[k] = reinterpret_cast<const u32x4_t*>(g)[tid + kT2 * k];
    };
    const auto fetch_hin = [&](int64_t h) {
        const u16* g = reinterpret_cast<const u16*>(p.hin) + state_at(h);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) hinf[ks] = *reinterpret_cast<const uint4*>(g + (16 * nt + r) * kP2 + ks * 32 + 8 * q);
    };
    // The walk over the heads is a pipeline with one barrier a head: while the
    // products of head h run, its workgroup stages x, dy and the factors of head
    // h + 2, evaluates the scores of h + 1, and finishes the per-token sums of
    // h - 1.  Each of these reads what an earlier step wrote and writes buffers
    // that nobody reads in this step: x, dy and the scores' sums lie in three
    // buffers (head mod 3), the scores, Gn and the other sums in two, the factors
    // in four.  Past the last head the early stages run on its inputs once more
    // (no branches: the compiler then counts the loads in flight); nobody reads
    // their results.
    const auto setup = [&](int64_t h, int x3, int k) {   // from the registers of fetch(h)
        u16* const xs = xs3 + kQ2 * kP2 * x3;
        u16* const dys = dys3 + kQ2 * kP2 * x3;
        float* const scs = scs4[k];
        float* const sdt = sdt4[k];
        float* const seend = seend4[k];
        float* const secs = secs4[k];
        // this head's x, dy (fetched during the previous head) into shared memory
        if constexpr (H32)
            pd = make_uint4(pack2(pf0.x, pf0.y), pack2(pf0.z, pf0.w), pack2(pf1.x, pf1.y), pack2(pf1.z, pf1.w));
        *reinterpret_cast<uint4*>(xs + staged) = px;
        *reinterpret_cast<uint4*>(dys + staged) = pd;
        if (w == 0) {
            // cumsum of dt*A (log2 units) and the per-token factors
            const float A2 = -expf(A_logp[h]) * kLog2e;
            const float dtv = dt_of_raw<H32>(pdt);
            const float cs = wave_scan(dtv * A2);
            const float csend = lane_value(cs, L - 1);
            scs[lane] = cs;
            sdt[lane] = dtv;
            seend[lane] = lane < L ? exp2f(csend - cs) : 0.f;
            secs[lane] = lane < L ? exp2f(cs) : 0.f;
        }
    };
    const auto store_gn = [&](int g2) {   // from the registers of fetch_gn
#pragma unroll
        for (int k = 0; k < N / 64; ++k)
            *reinterpret_cast<u32x4_t*>(Gn2 + kQ2 * N * g2 + kQ2 * kP2 * k + staged) = gpc[k];
    };
    const auto scores = [&](int x3, int g2, int k4) {
        const u16* const xs = xs3 + kQ2 * kP2 * x3;
        const u16* const dys = dys3 + kQ2 * kP2 * x3;
        u16* const Gs = Gs2 + kQ2 * kP2 * g2;
        u16* const Rs = Rs2 + kQ2 * kP2 * g2;
        const float* const scs = scs4[k4];
        const float* const sdt = sdt4[k4];
        auto& rowp = rowp3[x3];
        auto& colp = colp3[x3];
        const LaneOffs<N> o(lane, pw);
        const int r = o.r, q = o.q;
        // --- score tiles: R0 = dy x^T (then dt_t), Gs, Rs, l and their sums
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            if (k < ntile) {
                const int2 tl = kLowerTile[w + 2 * k];
                f32x4_t acc = zero4();
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
                    acc = mma(o.row64(dys, tl.x, ks), o.row64(xs, tl.y, ks), acc);
                const int t = 16 * tl.y + r, u0 = 16 * tl.x + 4 * q;
                const float dtt = sdt[t], cst = scs[t];
                const float4 csu = *reinterpret_cast<const float4*>(scs + u0);
                const float cu[4] = {csu.x, csu.y, csu.z, csu.w};
                float gs[4], rs[4], l[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const bool on = u0 + v >= t && u0 + v < L;
                    const float e = exp2f(cu[v] - cst);
                    const float r0 = acc[v] * dtt;
                    gs[v] = on ? e * g0[k][v] : 0.f;   // (not 0 times what may be infinite)
                    rs[v] = on ? e * r0 : 0.f;
                    l[v] = on ? gs[v] * r0 : 0.f;
                }
                const float rsum = row_sum16x4(l[0], l[1], l[2], l[3], r);
                if (r < 4) rowp[tl.y][u0 + r] = rsum;
                const float csum = col_sum4((l[0] + l[1]) + (l[2] + l[3]));
                if (q == 0) colp[tl.x][t] = csum;
                const int off = (tl.x >> 1 ? o.oa[1] : o.oa[0]) + 8 * (tl.x & 1) + 32 * kP2 * tl.y;
                *reinterpret_cast<uint2*>(reinterpret_cast<char*>(Gs) + off) = make_uint2(pack2(gs[0], gs[1]), pack2(gs[2], gs[3]));
                *reinterpret_cast<uint2*>(reinterpret_cast<char*>(Rs) + off) = make_uint2(pack2(rs[0], rs[1]), pack2(rs[2], rs[3]));
            }
        }
    };
    // wavefront 1; lane k holds token t = 63 - k, so that a prefix sum over lanes
    // is a suffix sum over tokens: dcs, then the decay gradients
    const auto per_token = [&](int64_t h, int x3, int g2, int k4) {
        const float* const sdt = sdt4[k4];
        const float* const seend = seend4[k4];
        const float* const secs = secs4[k4];
        const auto& rowp = rowp3[x3];
        const auto& colp = colp3[x3];
        const auto& xdp = xdp2[g2];
        const auto& q1p = q1p2[g2];
        const auto& ghp = ghp2[g2];
        const auto& dyxp = dyxp2[g2];
        const int64_t bh = b * p.H + h;
            const int t = kQ2 - 1 - lane;
            const bool in = t < L;
            float s2 = 0.f, row = 0.f, col = 0.f, s1 = 0.f, xd = 0.f;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                s2 += xdp[1][k][t];
                row += rowp[k][t];
                col += colp[k][t];
                xd += xdp[0][k][t];
            }
#pragma unroll
            for (int k = 0; k < kNT; ++k) s1 += q1p[k][t];
            const float q2 = in ? sdt[t] * s2 : 0.f;   // X~_t . (Gn B_t)
            const float ghs = wave_sum(lane < 32 ? ghp[lane & 31] : 0.f);
            const float hsum = wave_sum(seend[t] * q2);
            float dcs = in ? row - col + secs[t] * s1 - seend[t] * q2 : 0.f;
            if (t == L - 1) dcs += secs[t] * ghs + hsum;   // <Gn, h_out>
            const float da = wave_scan(dcs);   // over tokens t' >= t
            if (in) {
                const float g = fmaf(-expf(A_logp[h]), da, xd);
                if constexpr (H32)
                    static_cast<float*>(p.ddt)[(t0 + t) * p.H + h] = g;
                else
                    static_cast<u16*>(p.ddt)[(t0 + t) * p.H + h] = static_cast<u16>(bf16_bits(g));
            }
            const float sa = wave_sum(in ? sdt[t] * da : 0.f);
            const float sd = wave_sum(lane < 32 ? dyxp[lane & 31] : 0.f);
            if (lane == 0) {
                p.dAp[bh * p.nC + c] = sa;
                p.dDp[bh * p.nC + c] = sd;
            }
    };
    const auto clamp = [&](int64_t h) { return h < hr.hi ? h : hr.hi - 1; };
    fetch(hr.lo);
    fetch_gn(hr.lo);
    fetch_hin(hr.lo);
    setup(hr.lo, 0, 0);
    fetch(clamp(hr.lo + 1));
    setup(clamp(hr.lo + 1), 1, 1);
    fetch(clamp(hr.lo + 2));
    __syncthreads();
    store_gn(0);   // (over C, which all have read)
    fetch_gn(clamp(hr.lo + 1));
    scores(0, 0, 0);
    __syncthreads();
    int x0 = 0, x1 = 1, x2 = 2;   // buffers of heads h, h + 1, h + 2 (= h - 1)
    for (int64_t h = hr.lo; h < hr.hi; ++h) {
        const int k = static_cast<int>(h - hr.lo), g2 = k & 1, k4 = k & 3;
        setup(clamp(h + 2), x2, (k + 2) & 3);
        fetch(clamp(h + 3));
        store_gn(g2 ^ 1);
        fetch_gn(clamp(h + 2));
        scores(x1, g2 ^ 1, (k + 1) & 3);

        const float Dh = Dp ? Dp[h] : 0.f;
        const u16* const xs = xs3 + kQ2 * kP2 * x0;
        const u16* const dys = dys3 + kQ2 * kP2 * x0;
        const u16* const Gs = Gs2 + kQ2 * kP2 * g2;
        const u16* const Rs = Rs2 + kQ2 * kP2 * g2;
        const u16* const Gn = Gn2 + kQ2 * N * g2;
        const float* const sdt = sdt4[k4];
        const float* const seend = seend4[k4];
        const float* const secs = secs4[k4];
        auto& xdp = xdp2[g2];
        auto& q1p = q1p2[g2];
        auto& ghp = ghp2[g2];
        auto& dyxp = dyxp2[g2];
        // --- dX~^T (p x t): dy^T Gs + e(end,t) Gn B^T; dx, and per-token sums.  P-tile
        // w % 4, token tiles w / 4 and w / 4 + 2 (whose scores with u < 32 are zero)
        float sxd[2], sxg[2], sdx = 0.f;
        const LaneOffs<N> o(lane, pw);
        const int r = o.r, q = o.q, p0 = 16 * pw + 4 * q;
        {
            float4 d32[2];
            if constexpr (H32) {   // (read by the fetch three heads before, where it was rounded)
                const __amdgpu_buffer_rsrc_t rd = __builtin_amdgcn_make_buffer_rsrc(
                    const_cast<float*>(static_cast<const float*>(p.dy)) + (t0 * p.H + h) * kP2, 0,
                    ((L - 1) * xrow + kP2) * 4, 0x00020000);
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    d32[j] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(
                                                            rd, ((16 * ((w >> 2) + 2 * j) + r) * xrow + p0) * 4, 0, 0));
            }
            // (rows past a partial chunk are dropped by the buffer bounds: no branch)
            const __amdgpu_buffer_rsrc_t rdx = __builtin_amdgcn_make_buffer_rsrc(
                static_cast<u16*>(p.dx) + (t0 * p.H + h) * kP2, 0,
                ((L - 1) * xrow + kP2) * static_cast<int>(sizeof(u16)), 0x00020000);
            f32x4_t ai[2], ag[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) ai[j] = ag[j] = zero4();
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                const uint4 a = o.tr64(dys, ks, o.ot);
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    if (j == 0 || ks == 1) ai[j] = mma(a, o.row64(Gs, (w >> 2) + 2 * j, ks), ai[j]);
            }
#pragma unroll
            for (int ks = 0; ks < N / 32; ++ks) {
                const uint4 a = o.tr64(Gn, ks, o.ot);
#pragma unroll
                for (int j = 0; j < 2; ++j) ag[j] = mma(a, o.rowN(Bs, (w >> 2) + 2 * j, ks), ag[j]);
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int t = 16 * ((w >> 2) + 2 * j) + r;
                const float ee = seend[t], dtt = sdt[t];
                const uint2 xv = *reinterpret_cast<const uint2*>(o.at(xs, 32 * kP2 * ((w >> 2) + 2 * j) + o.ox));
                const float xf[4] = {lo_f(xv.x), hi_f(xv.x), lo_f(xv.y), hi_f(xv.y)};
                float df[4];
                if constexpr (H32) {
                    df[0] = d32[j].x; df[1] = d32[j].y; df[2] = d32[j].z; df[3] = d32[j].w;
                } else {
                    const uint2 dv = *reinterpret_cast<const uint2*>(o.at(dys, 32 * kP2 * ((w >> 2) + 2 * j) + o.ox));
                    df[0] = lo_f(dv.x); df[1] = hi_f(dv.x); df[2] = lo_f(dv.y); df[3] = hi_f(dv.y);
                }
                float dx[4];
                sxd[j] = sxg[j] = 0.f;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float dX = fmaf(ee, ag[j][v], ai[j][v]);
                    dx[v] = fmaf(dtt, dX, Dh * df[v]);
                    sxd[j] = fmaf(xf[v], dX, sxd[j]);
                    sxg[j] = fmaf(xf[v], ag[j][v], sxg[j]);
                    sdx = fmaf(df[v], xf[v], sdx);
                }
                __builtin_amdgcn_raw_buffer_store_b64(u32x2_t{pack2(dx[0], dx[1]), pack2(dx[2], dx[3])}, rdx,
                                                      (t * xrow + p0) * static_cast<int>(sizeof(u16)), 0, 0);
            }
        }
        // (lane group q: x . dX~ and x . (Gn B) of the first and the second token tile)
        xdp[q >> 1][pw][16 * ((w >> 2) + 2 * (q & 1)) + r] = col_sum4x4(sxd[0], sxd[1], sxg[0], sxg[1]);
        sdx = row_sum16(sdx);
        if (r == 0) dyxp[4 * w + q] = sdx;

        // --- dB^T (n x t) += C^T Rs + e(end,t) dt_t Gn^T x^T
        uint4 gntf[2];
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) gntf[ks] = o.row64(Gn, nt, ks);
#pragma unroll
        for (int j = 0; j < kBW; ++j) {
            const int tt = tile_of(j);
            f32x4_t bx = zero4();
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                if (j < kBW / 2 || ks == 1)   // (token tiles 2 and 3: no u < 32)
                    dBacc[j] = mma(ctf[ks], o.row64(Rs, tt, ks), dBacc[j]);
                bx = mma(gntf[ks], o.row64(xs, tt, ks), bx);
            }
            const float fb = seend[16 * tt + r] * sdt[16 * tt + r];
#pragma unroll
            for (int v = 0; v < 4; ++v) dBacc[j][v] = fmaf(fb, bx[v], dBacc[j][v]);
        }
        // --- dC^T (n x u) += B^T Rs^T + exp(cs_u) h_in^T dy^T, and dy_u . (h_in C_u)
        float q1[kBW];
#pragma unroll
        for (int j = 0; j < kBW; ++j) {
            const int tt = tile_of(j);
            f32x4_t ch = zero4();
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                if (j >= kBW / 2 || ks == 0)   // (token tiles 0 and 1: no t >= 32)
                    dCacc[j] = mma(btf[ks], o.tr64(Rs, ks, o.op[kBW == 4 ? j >> 1 : j] + 8 * (tt & 1)), dCacc[j]);
                ch = mma(hinf[ks], o.row64(dys, tt, ks), ch);
            }
            const float fc = secs[16 * tt + r];
            asm volatile("" : "+v"(cv[j].x), "+v"(cv[j].y));   // (kept packed across the heads)
            const float cf[4] = {lo_f(cv[j].x), hi_f(cv[j].x), lo_f(cv[j].y), hi_f(cv[j].y)};
            q1[j] = 0.f;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                dCacc[j][v] = fmaf(fc, ch[v], dCacc[j][v]);
                q1[j] = fmaf(cf[v], ch[v], q1[j]);
            }
        }
        {   // lane group q gets the sum of token tile tile_of(q)
            const float s = col_sum4x4(q1[0], q1[1], q1[kBW - 2], q1[kBW - 1]);
            if (q < kBW) q1p[nt][16 * tile_of(q) + r] = s;
        }
        {
            // <Gn, h_in>: the diagonal of Gn^T (h_in^T)^T over this wavefront's n-tile
            // (with dstate 64 two wavefronts hold each tile, the even one counts it)
            f32x4_t d = zero4();
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) d = mma(gntf[ks], hinf[ks], d);
            float gh = (r & 2) ? ((r & 1) ? d[3] : d[2]) : ((r & 1) ? d[1] : d[0]);
            gh = r >> 2 == q && (kBW == 4 || (w & 1) == 0) ? gh : 0.f;
            gh = row_sum16(gh);
            if (r == 0) ghp[4 * w + q] = gh;
        }
        fetch_hin(clamp(h + 1));
        if (w == 1 && h > hr.lo) per_token(h - 1, x2, g2 ^ 1, (k + 3) & 3);
        __syncthreads();
        const int t = x0;
        x0 = x1;
        x1 = x2;
        x2 = t;
    }
    if (w == 1) {
        const int k = static_cast<int>(hr.hi - 1 - hr.lo);
        per_token(hr.hi - 1, x2, k & 1, k & 3);
    }

    // this slice's dB and dC for the chunk: lane holds n = 16 nt + 4 q + v, t = 16 tt + r.
    // With one slice per group these sums are the gradients: rounded here to
    // bf16 (nearest even, as the reduction over slices rounds them) and stored
    // in place, and the launch skips that reduction (bc_direct).
#pragma unroll
    for (int j = 0; j < kBW; ++j) {
        const int t = 16 * tile_of(j) + r;
        if (t < L) {
            if constexpr (DIRECT) {
                const int64_t o = ((t0 + t) * p.G + hr.g) * N + 16 * nt + 4 * q;
                *reinterpret_cast<uint2*>(static_cast<u16*>(p.dB) + o) =
                    make_uint2(pack2(dBacc[j][0], dBacc[j][1]), pack2(dBacc[j][2], dBacc[j][3]));
                *reinterpret_cast<uint2*>(static_cast<u16*>(p.dC) + o) =
                    make_uint2(pack2(dCacc[j][0], dCacc[j][1]), pack2(dCacc[j][2], dCacc[j][3]));
            } else {
                const int64_t o = ((hr.slice * p.b * p.T + t0 + t) * p.G + hr.g) * N + 16 * nt + 4 * q;
                *reinterpret_cast<float4*>(p.dBp + o) =
                    make_float4(dBacc[j][0], dBacc[j][1], dBacc[j][2], dBacc[j][3]);
                *reinterpret_cast<float4*>(p.dCp + o) =
                    make_float4(dCacc[j][0], dCacc[j][1], dCacc[j][2], dCacc[j][3]);
            }
        }
    }
}

template <int N, bool PACKED, bool H32, bool DIRECT>
hipError_t launch_chunk(const BwdParams& p, dim3 grid, size_t sm, hipStream_t st)
{
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_bwd2_chunk<N, PACKED, H32, DIRECT>),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(sm));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_bwd2_chunk<N, PACKED, H32, DIRECT>), grid, dim3(kT2), sm, st, p, p.A_log, p.D);
    return hipGetLastError();
}

template <int N>
hipError_t launch_fast(const BwdParams& params, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1)
{
    BwdParams p = params;
    p.bc_direct = p.S == 1 && reinterpret_cast<uintptr_t>(p.dB) % 8 == 0 && reinterpret_cast<uintptr_t>(p.dC) % 8 == 0;
    const bool packed = p.vtab != nullptr, h32 = p.h32 != 0, direct = p.bc_direct != 0;
    if (packed && h32) return hipErrorInvalidValue;   // float32 handoffs: plain rows only
    const size_t sm_chunk = chunk_smem<N>();
    hipError_t e;
    if (packed)   // one workgroup per (sequence, head) and direction
        hipLaunchKernelGGL((k_bwd2_pass<N, true, false>), dim3(static_cast<unsigned>(p.nseq * p.H), 2), dim3(kPassT),
                           0, st, p);
    else if (h32)
        hipLaunchKernelGGL((k_bwd2_pass<N, false, true>), dim3(static_cast<unsigned>(p.b * p.H), 2), dim3(kPassT), 0,
                           st, p);
    else
        hipLaunchKernelGGL((k_bwd2_pass<N, false, false>), dim3(static_cast<unsigned>(p.b * p.H), 2), dim3(kPassT), 0,
                           st, p);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (ev0 && (e = hipEventRecord(ev0, st)) != hipSuccess) return e;
    const dim3 grid(static_cast<unsigned>(p.nC), static_cast<unsigned>(p.b), static_cast<unsigned>(p.G * p.S));
    if (packed)
        e = direct ? launch_chunk<N, true, false, true>(p, grid, sm_chunk, st)
                   : launch_chunk<N, true, false, false>(p, grid, sm_chunk, st);
    else if (h32)
        e = direct ? launch_chunk<N, false, true, true>(p, grid, sm_chunk, st)
                   : launch_chunk<N, false, true, false>(p, grid, sm_chunk, st);
    else
        e = direct ? launch_chunk<N, false, false, true>(p, grid, sm_chunk, st)
                   : launch_chunk<N, false, false, false>(p, grid, sm_chunk, st);
    if (e != hipSuccess) return e;
    if (ev1 && (e = hipEventRecord(ev1, st)) != hipSuccess) return e;
    return launch_backward_reduce(p, true, st, !direct);
}

}  // namespace

bool bwd_fast_supported(bool bf16, int64_t P, int64_t N) { return bf16 && P == kP2 && (N == 64 || N == 128); }

hipError_t launch_backward_fast(const BwdParams& p, hipStream_t stream, hipEvent_t ev_begin, hipEvent_t ev_end)
{
    return p.N == 64 ? launch_fast<64>(p, stream, ev_begin, ev_end) : launch_fast<128>(p, stream, ev_begin, ev_end);
}

}  // namespace ssd

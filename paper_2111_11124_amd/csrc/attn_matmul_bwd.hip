// attn_matmul_bwd.hip -- backward of the two matrix products of self-attention at head-wise
// de-quantized operands (Sec. 3.1 Eq. 2 with G_l the gradient of a matrix product; Sec. 3.2: the
// operands of the products are saved as 8-bit codes with one (alpha, beta) pair per head):
//   O = A V           dA[i,j] = sum_d dO[i,d]*V_hat[j,d]           dV[j,d] = sum_i A_hat[i,j]*dO[i,d]
//   S = scale Q K^T   dQ[i,d] = scale*sum_j dS[i,j]*K_hat[j,d]     dK[j,d] = scale*sum_i dS[i,j]*Q_hat[i,d]
//
// All four are one batched product  C[r,c] = sum_t P(r,t)*Q(t,c)  per (sample, head), where P and Q are
// strided views of the tensors and exactly one of them is coded.  As in the weight gradient, the matrix
// cores contract with the signed codes themselves (exact in binary16) and the head's affine map is
// applied to the finished sums:  x_hat = s*(q+128) + beta  gives
//   C = s * sum_t P*q  +  (beta + 128 s) * sum_t P        (Q coded; symmetric when P is),
// the plain sums coming from one more MFMA against a fragment of ones.
//
// The sequence length of a vision transformer is odd (197), so rows of the attention-shaped tensors
// start at odd offsets and nothing here can be loaded in ALIGNED vectors: operand tiles of 64 x 32 are
// staged into LDS with element-aligned 8-element loads along each operand's unit-stride index (whole
// vectors inside the extents, single elements and zero fill at the edges, so any extents work) and
// kept in the operand's own orientation; where that is not the orientation the MFMA wants, the
// fragments come from the LDS transpose reads.  The next stage's loads are in flight while a stage
// is multiplied.  binary16 or bfloat16 tensors (every kernel here takes the number type as a parameter);
// binary32 tensors run the general kernel, or the one for few heads, on three bfloat16 parts.
//
// That general kernel (k_bmm_q) serves every shape; few heads go to k_bmm_waves (bmm_waves), a launch with both of a call's products;
// dedicated kernels take over where there is work enough for them (da_way, tn_way,
// nn_way): k_attn_da, k_attn_tn, k_attn_nn for sequences that one workgroup per head (or per 32 rows) holds, odd lengths
// included, and k_attn_da_cols, k_attn_tn_cols, k_attn_nn_rows, by tiles, for sequences of any length from 64 on (a pitch of N elements
// with N a multiple of 32 puts the first three kernels' lanes on the same LDS banks).  The tile kernels' rows may start at any
// element (ANY): a vector that is not aligned touches one cache line more, and from LDS on everything is aligned.  Whole backward (four
// products), general kernel -> by tiles: (16, 12, 577, 64) 182 -> 129 us, (8, 8, 919, 64) 151 -> 101, (64, 6, 301, 96) 182 -> 105.
#include <hip/hip_runtime.h>
#include <type_traits>

#include "api_util.hpp"
#include "common.hpp"

namespace mesa {

typedef _Float16 bm_v8h __attribute__((ext_vector_type(8)));
typedef _Float16 bm_v2h __attribute__((ext_vector_type(2)));
typedef _Float16 bm_v4h __attribute__((ext_vector_type(4)));
typedef short bm_v4s __attribute__((ext_vector_type(4)));
typedef int bm_v2i __attribute__((ext_vector_type(2)));
typedef float bm_v16f __attribute__((ext_vector_type(16)));
typedef float bm_v4f __attribute__((ext_vector_type(4)));
typedef unsigned bm_v4u __attribute__((ext_vector_type(4)));

#define BM_LDS3(T, p) ((__attribute__((address_space(3))) T *)(p))

constexpr int kBmTile = 64;     // output tile of a workgroup (rows and columns)
constexpr int kBmT = 32;        // contraction extent per stage
constexpr int kBmParts = kBmT / 32;   // 8-element vectors per thread, operand and stage

// eight signed codes (bytes) -> eight binary16 values q: 0x6400 | (byte ^ 0x80) is 1152 + q exactly
__device__ __forceinline__ bm_v8h bm_codes_to_half8(bm_v2i raw)
{
    bm_v8h out;
    const h2 k1152 = {(_Float16)1152.0f, (_Float16)1152.0f};
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        const uint32_t x = uint32_t(raw[w]) ^ 0x80808080u;
        const h2 lo = as_h2(__builtin_amdgcn_perm(0x64646464u, x, 0x04010400u)) - k1152;   // bytes 0, 1
        const h2 hi = as_h2(__builtin_amdgcn_perm(0x64646464u, x, 0x04030402u)) - k1152;   // bytes 2, 3
        out[4 * w + 0] = lo.x; out[4 * w + 1] = lo.y; out[4 * w + 2] = hi.x; out[4 * w + 3] = hi.y;
    }
    return out;
}

// What the 16-bit number type decides in the general kernel: how codes become matrix-core operands and which
// value of the code is contracted (kCentre: c in "operand = x_bar - c"; bfloat16 has no spare mantissa bit for
// the exponent trick and takes x_bar = q + 128 itself, byte -> binary32 -> upper half), the fragment of ones,
// the MFMA and the rounding of a result.  Operands travel as raw 16-bit lanes (bm_v8h as a container).
typedef __bf16 bm_v8b __attribute__((ext_vector_type(8)));
template <typename ET> struct BmNum;
template <> struct BmNum<_Float16> {
    static constexpr float kCentre = 128.0f;
    static constexpr uint16_t kOne = 0x3C00u;
    __device__ static __forceinline__ bm_v8h codes8(bm_v2i raw) { return bm_codes_to_half8(raw); }
    __device__ static __forceinline__ bm_v16f mfma(bm_v8h a, bm_v8h b, bm_v16f c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
    }
    __device__ static __forceinline__ _Float16 round(float v) { return (_Float16)v; }
    // eight codes gathered two to a register (bits 0-7 and 16-23): 0x6400 | (byte ^ 0x80) is 1024 + x_bar, minus 1152
    __device__ static __forceinline__ bm_v8h gathered(bm_v4u u)
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) u[k] = (u[k] ^ 0x00800080u) | 0x64006400u;
        bm_v8h f = __builtin_bit_cast(bm_v8h, u);
#pragma unroll
        for (int k = 0; k < 8; ++k) f[k] = f[k] - (_Float16)1152.0f;
        return f;
    }
    // acc + the two values of a register pair
    __device__ static __forceinline__ float dot_ones(_Float16 a, _Float16 b, float acc)
    {
        return __builtin_amdgcn_fdot2(bm_v2h{a, b}, bm_v2h{(_Float16)1.0f, (_Float16)1.0f}, acc, false);
    }
};
template <> struct BmNum<__bf16> {
    static constexpr float kCentre = 0.0f;
    static constexpr uint16_t kOne = 0x3F80u;
    __device__ static __forceinline__ bm_v8h codes8(bm_v2i raw)
    {
        bm_v4u out;
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const uint32_t x = uint32_t(raw[w]) ^ 0x80808080u;
            const uint32_t f0 = __float_as_uint(float(x & 0xFFu)), f1 = __float_as_uint(float((x >> 8) & 0xFFu));
            const uint32_t f2 = __float_as_uint(float((x >> 16) & 0xFFu)), f3 = __float_as_uint(float(x >> 24));
            out[2 * w] = __builtin_amdgcn_perm(f1, f0, 0x07060302u);
            out[2 * w + 1] = __builtin_amdgcn_perm(f3, f2, 0x07060302u);
        }
        return __builtin_bit_cast(bm_v8h, out);
    }
    __device__ static __forceinline__ bm_v16f mfma(bm_v8h a, bm_v8h b, bm_v16f c)
    {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bm_v8b, a), __builtin_bit_cast(bm_v8b, b), c, 0, 0, 0);
    }
    __device__ static __forceinline__ _Float16 round(float v)   // the bits of the bfloat16, in the 16-bit container
    {
        return __builtin_bit_cast(_Float16, __bf16(v));
    }
    __device__ static __forceinline__ bm_v8h gathered(bm_v4u u)
    {
        bm_v4u out;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t x = u[k] ^ 0x00800080u;
            out[k] = __builtin_amdgcn_perm(__float_as_uint(float((x >> 16) & 0xFFu)), __float_as_uint(float(x & 0xFFu)), 0x07060302u);
        }
        return __builtin_bit_cast(bm_v8h, out);
    }
    __device__ static __forceinline__ float dot_ones(_Float16 a, _Float16 b, float acc)
    {
        typedef __bf16 v2b __attribute__((ext_vector_type(2)));
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(v2b, bm_v2h{a, b}), __builtin_bit_cast(v2b, 0x3F803F80u), acc, false);
    }
};

// binary32 tensors: 2^23 times a binary32 value is exactly the sum of three bfloat16 values (cut_f32), a code q is exact in
// bfloat16 and a product of the two in binary32, so three bfloat16 MFMAs add the same exact products as the binary32
// MFMA, at sixteen times its rate and with one rounding of the sum per sixteen steps instead of per two.  A workgroup that met
// a value of 2^64 or more, or an infinity, does its tile again with binary32 MFMAs, as the plain kernel does.  The contracted value is the signed code, as in the plain binary32 kernel.  Against that kernel (one element
// per lane and load, straight from memory, a dependent load per two contraction steps) the four products and softmax's
// backward took 140 -> 45 us at (2, 3, 197, 64), 257 -> 62 at (1, 12, 324, 64) and 312 -> 93 at (32, 6, 197, 64).
template <> struct BmNum<float> {
    static constexpr float kCentre = 128.0f;
    static constexpr uint16_t kOne = 0x3F80u;
    __device__ static __forceinline__ bm_v8h codes8(bm_v2i raw)
    {
        bm_v4u out;
#pragma unroll
        for (int w = 0; w < 2; ++w) {
            const int x = raw[w];
            const uint32_t f0 = __float_as_uint(float(int(int8_t(x)))), f1 = __float_as_uint(float(int(int8_t(x >> 8))));
            const uint32_t f2 = __float_as_uint(float(int(int8_t(x >> 16)))), f3 = __float_as_uint(float(x >> 24));
            out[2 * w] = __builtin_amdgcn_perm(f1, f0, 0x07060302u);
            out[2 * w + 1] = __builtin_amdgcn_perm(f3, f2, 0x07060302u);
        }
        return __builtin_bit_cast(bm_v8h, out);
    }
    __device__ static __forceinline__ bm_v16f mfma(bm_v8h a, bm_v8h b, bm_v16f c) { return BmNum<__bf16>::mfma(a, b, c); }
    __device__ static __forceinline__ float round(float v) { return v; }
};

// Workgroups b, b + 8, .. run on one XCD: the number that gives each XCD a run of neighbouring pieces of work (they share operands in its
// L2).  A permutation of 0 .. total-1.
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned total)
{
    const unsigned x = b % 8u, q = total / 8u, r = total % 8u;
    return x * q + (x < r ? x : r) + b / 8u;
}

// the 16 bytes of v moved down by 0 .. 15 bytes, zeros above them
__device__ __forceinline__ u32x4 move_down(u32x4 v, int bytes)
{
    if (bytes & 8) v = u32x4{v[2], v[3], 0u, 0u};
    if (bytes & 4) v = u32x4{v[1], v[2], v[3], 0u};
    const uint32_t r = uint32_t(bytes) & 3u;
    return u32x4{__builtin_amdgcn_alignbyte(v[1], v[0], r), __builtin_amdgcn_alignbyte(v[2], v[1], r), __builtin_amdgcn_alignbyte(v[3], v[2], r),
                 __builtin_amdgcn_alignbyte(0u, v[3], r)};
}

struct BmmArgs {
    const _Float16 *x;          // the plain operand (16-bit container: binary16 or bfloat16 bits; k_bmm_q<float>: binary32)
    const int8_t *y;            // the coded operand
    _Float16 *c;                // output, row-major R x Cn per batch (of the plain operand's type)
    int64_t x_batch, y_batch, c_batch;   // elements per (sample, head)
    int R, Cn, Tn;              // output rows, output columns, contraction extent
    int64_t p_rs, p_ts;         // element strides of the view P(r, t)
    int64_t q_ts, q_cs;         // element strides of the view Q(t, c)
    int tiles_r, tiles_c;
    int64_t batch0;             // first (sample, head) of this launch
    int head0;                  // and its head: batch0 % heads
    int heads;
    float scale;
    const float *alpha, *beta;  // of the coded operand, per head
};

// ---- staging: global -> registers -> LDS ---------------------------------------------------------
// A 64 x kBmT operand tile per stage is kBmParts * 256 vectors of eight elements along the operand's
// unit-stride index (vector idx = tid + 256 * part), each loaded with one element-aligned 16-byte
// (binary16) or 8-byte (codes) load and stored to LDS as it is, in the operand's own orientation:
//   TFAST  (unit stride along the contraction index t):  idx -> (line = idx / (kBmT/8), t = 8 * (idx % (kBmT/8)) ..+7),
//          LDS rows are lines ([line][t]) and an MFMA fragment is a plain 16- or 8-byte read;
//   !TFAST (unit stride along the row / column index):   idx -> (t = idx/8, lines 8*(idx%8) ..+7),
//          LDS rows are contraction steps ([t][line]) and the fragment comes from gfx950's transposing
//          LDS reads (ds_read_b64_tr_b16 / _b8: within 16 lanes, the lanes 4k..4k+3 -- 2k, 2k+1 for bytes --
//          supply row k, and lane i receives column i).
// `line` is the row of P or the column of Q.  Codes stay bytes in LDS and become binary16 (the signed
// code itself, exact) in the fragment.  Row pitches are padded so that neither access conflicts.
//
// binary32 (ET = float): eight elements are two 16-byte loads; the store cuts them into kPlanes = 3 bfloat16 parts, each a
// tile of its own in LDS that is read like a 16-bit operand's.
template <bool CODED, typename ET> struct BmElem {   // plain 16-bit operand
    typedef _Float16 global_t, lds_t;
    typedef u32x4 raw_t;        // eight elements as loaded
    typedef u32x4 word_t;       // and as they lie in LDS
    static constexpr int kEb = 2, kPlanes = 1;
    __device__ static __forceinline__ void cut(const raw_t &v, word_t (&w)[kPlanes]) { w[0] = v; }
};
template <typename ET> struct BmElem<true, ET> {     // codes
    typedef int8_t global_t, lds_t;
    typedef u32x2 raw_t, word_t;
    static constexpr int kEb = 1, kPlanes = 1;
    __device__ static __forceinline__ void cut(const raw_t &v, word_t (&w)[kPlanes]) { w[0] = v; }
};
template <> struct BmElem<false, float> {
    typedef float global_t;
    typedef _Float16 lds_t;     // bfloat16 bits
    struct raw_t { u32x4 lo, hi; };
    typedef u32x4 word_t;
    static constexpr int kEb = 2, kPlanes = 3;
    __device__ static __forceinline__ void cut(const raw_t &v, word_t (&w)[kPlanes])
    {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            uint32_t part[3][2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                cut_f32(__uint_as_float(k < 2 ? v.lo[2 * k + j] : v.hi[2 * k - 4 + j]), part[0][j], part[1][j], part[2][j]);
            }
#pragma unroll
            for (int q = 0; q < 3; ++q) w[q][k] = __builtin_amdgcn_perm(part[q][1], part[q][0], 0x07060302u);
        }
    }
    // the largest magnitude, of m or an element
    __device__ static __forceinline__ float most(float m, const raw_t &v)
    {
#pragma unroll
        for (int k = 0; k < 4; k += 2) {
            m = max_magnitude(m, __uint_as_float(v.lo[k]), __uint_as_float(v.lo[k + 1]));
            m = max_magnitude(m, __uint_as_float(v.hi[k]), __uint_as_float(v.hi[k + 1]));
        }
        return m;
    }
};

// Edges.  Rows of P / columns of Q beyond the extents produce output rows / columns that are never
// written, so they may hold any finite data; contraction steps t >= Tn must contribute nothing, so both
// operands hold zeros there (never stale LDS contents: 0 x NaN would poison a sum).  Every load is an
// unconditional whole-vector load from coordinates clamped into the tensor (no branch, no merge with
// other values: nothing waits on a load before its stage is due); a vector that was moved back to stay
// inside the extent is written to LDS at the position it really came from (element by element: the
// slots overlap the neighbouring vector's, with the same values), and zeros are written where required.
template <bool CODED, bool TFAST, typename ET> struct BmOperand {
    typedef BmElem<CODED, ET> Elem;
    typedef typename Elem::global_t E;
    typedef typename Elem::lds_t L;
    typedef typename Elem::raw_t Raw;
    typedef typename Elem::word_t W;
    static constexpr int kEb = Elem::kEb, kPlanes = Elem::kPlanes;
    // bytes per LDS row: [line][t]: kBmT elements + 8 of padding; [t][line]: 64 elements + 32 of padding
    static constexpr int kPitch = TFAST ? (kBmT + 8) * kEb : (kBmTile + 32) * kEb;
    static constexpr int kPlane = TFAST ? kBmTile * kPitch : kBmT * kPitch;
    static constexpr int kBytes = kPlanes * kPlane;

    // tile-relative coordinates of vector idx: (line, t) of its first element
    __device__ static __forceinline__ void coord(int idx, int &line, int &t)
    {
        if (TFAST) { line = idx / (kBmT / 8); t = (idx % (kBmT / 8)) * 8; }
        else { t = idx / 8; line = (idx % 8) * 8; }
    }
    // lines >= 8 and tn >= 8 (checked by the entry points)
    __device__ static __forceinline__ Raw load(const E *base, int64_t line_stride, int64_t t_stride, int line0, int t0,
                                                        int lines, int tn, int idx)
    {
        int line, t;
        coord(idx, line, t);
        line += line0;
        t += t0;
        Raw v;
        if (TFAST) {
            line = line < lines ? line : lines - 1;
            t = t + 8 <= tn ? t : tn - 8;
            __builtin_memcpy(&v, base + int64_t(line) * line_stride + t, 8 * sizeof(E));       // t_stride == 1
        } else {
            t = t < tn ? t : tn - 1;
            line = line + 8 <= lines ? line : lines - 8;
            __builtin_memcpy(&v, base + int64_t(t) * t_stride + line, 8 * sizeof(E));          // line_stride == 1
        }
        return v;
    }
    __device__ static __forceinline__ void store(unsigned char *lds, const Raw &v, int line0, int t0, int lines, int tn, int idx)
    {
        W w[kPlanes];
        Elem::cut(v, w);
#pragma unroll
        for (int q = 0; q < kPlanes; ++q) store_plane(lds + q * kPlane, w[q], line0, t0, lines, tn, idx);
    }
    __device__ static __forceinline__ void store_plane(unsigned char *lds, const W &w, int line0, int t0, int lines, int tn, int idx)
    {
        int line, t;
        coord(idx, line, t);
        if (line0 + kBmTile <= lines && t0 + kBmT <= tn) {   // uniform: the whole tile lies inside the extents
            *reinterpret_cast<W *>(lds + (TFAST ? line * kPitch + t * kEb : t * kPitch + line * kEb)) = w;
            return;
        }
        L e[8];
        __builtin_memcpy(e, &w, sizeof(W));
        W zero;
#pragma unroll
        for (int k = 0; k < int(sizeof(W) / 4); ++k) zero[k] = 0u;
        if (TFAST) {
            unsigned char *row = lds + line * kPitch;
            const int tg = t0 + t;                                   // global contraction index of slot t
            if (tg + 8 <= tn) {
                *reinterpret_cast<W *>(row + t * kEb) = w;
            } else if (tg < tn) {                                    // the vector was moved back to tn - 8
                const int tc = tn - 8 - t0;                          // tile-relative slot of its first element (>= -7)
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (tc + i >= t) reinterpret_cast<L *>(row)[tc + i] = e[i];
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    if (tg + j >= tn) reinterpret_cast<L *>(row)[t + j] = L(0);
            } else {
                *reinterpret_cast<W *>(row + t * kEb) = zero;
            }
        } else {
            unsigned char *row = lds + t * kPitch;
            const bool t_ok = t0 + t < tn;
            const int lg = line0 + line;
            if (lg + 8 <= lines || lg >= lines) {                    // whole vector inside, or wholly outside (anything will do)
                *reinterpret_cast<W *>(row + line * kEb) = t_ok ? w : zero;
            } else {                                                 // moved back to lines - 8
                const int lc = lines - 8 - line0;
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (lc + i >= line) reinterpret_cast<L *>(row)[lc + i] = t_ok ? e[i] : L(0);
            }
        }
    }
    // the MFMA operand of a wave's 32 lines starting at l0, contraction slots 16*ks ..+15: lane l holds line
    // l%32 and the eight slots 8*(l/32) ..+7
    __device__ static __forceinline__ bm_v8h frag(const unsigned char *lds, int l0, int ks, int lane)
    {
        if (TFAST) {
            const unsigned char *p = lds + (l0 + (lane & 31)) * kPitch + (ks * 16 + (lane >> 5) * 8) * kEb;
            if (CODED) return BmNum<ET>::codes8(*reinterpret_cast<const bm_v2i *>(p));
            return *reinterpret_cast<const bm_v8h *>(p);
        }
        const int blk = lane >> 4, sl = lane & 15;
        if (CODED) {
            const unsigned char *p = lds + (ks * 16 + (blk >> 1) * 8 + (sl >> 1)) * kPitch + l0 + (blk & 1) * 16 + (sl & 1) * 8;
            return BmNum<ET>::codes8(__builtin_amdgcn_ds_read_tr8_b64_v2i32(BM_LDS3(bm_v2i, p)));
        }
        const unsigned char *p = lds + (ks * 16 + (blk >> 1) * 8 + (sl >> 2)) * kPitch + (l0 + (blk & 1) * 16 + (sl & 3) * 4) * 2;
        const bm_v4h lo = __builtin_bit_cast(bm_v4h, __builtin_amdgcn_ds_read_tr16_b64_v4i16(BM_LDS3(bm_v4s, p)));
        const bm_v4h hi = __builtin_bit_cast(bm_v4h, __builtin_amdgcn_ds_read_tr16_b64_v4i16(BM_LDS3(bm_v4s, p + 4 * kPitch)));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    }
};

// One wave's 32 x 32 tile with 32x32x2 binary32 MFMAs, operands straight from global memory, one element at a time (a lane needs
// one value per operand and step: lane l holds row r / column c, both l%32 of the tile, at contraction slot l/32).
// acc: the sums with the signed codes, acc1: those of the plain operand alone.  T: the tensors' element type.
template <bool P_CODED, typename T>
__device__ __forceinline__ void bmm_plain_sums(const BmmArgs &a, uint32_t b, int r, int c, bm_v16f &acc, bm_v16f &acc1)
{
    const int lane = threadIdx.x & 63;
    const int64_t xb0 = (int64_t(b) + a.batch0) * a.x_batch;
    const int8_t *yb = a.y + (int64_t(b) + a.batch0) * a.y_batch;
    const bool r_ok = r < a.R, c_ok = c < a.Cn;
#pragma unroll
    for (int v = 0; v < 16; ++v) { acc[v] = 0.0f; acc1[v] = 0.0f; }
    for (int t0 = 0; t0 < a.Tn; t0 += 2) {
        const int t = t0 + (lane >> 5);
        const bool t_ok = t < a.Tn;
        float pa = 0.0f, qb = 0.0f;
        const int64_t po = int64_t(r) * a.p_rs + int64_t(t) * a.p_ts, qo = int64_t(t) * a.q_ts + int64_t(c) * a.q_cs;
        if (t_ok && r_ok) pa = P_CODED ? float(int(yb[po])) : Store<T>::load1(a.x, xb0 + po);
        if (t_ok && c_ok) qb = P_CODED ? Store<T>::load1(a.x, xb0 + qo) : float(int(yb[qo]));
        const float one = t_ok ? 1.0f : 0.0f;
        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(pa, qb, acc, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_32x32x2f32(P_CODED ? one : pa, P_CODED ? qb : one, acc1, 0, 0, 0);   // sums of the plain operand
    }
}

// P_CODED: P is the coded operand (else Q).  P_TFAST / Q_TFAST: the contraction index is the unit-stride
// index of that operand in memory.  ET: the tensors' type (BmmArgs carries their pointers as 16-bit containers'; a
// binary32 operand is three bfloat16 planes, see BmElem).
// RS: groups of four waves that share out the contraction's stages (group g takes stages g, g + RS, ...), each with LDS tiles
// of its own; their sums are added through LDS at the end, in group order.  A stage behind the last one is all zeros
// (BmOperand::store).  For few workgroups with many stages: one workgroup's next stage is all that a CU has on its way.
template <bool P_CODED, bool P_TFAST, bool Q_TFAST, typename ET, int RS>
__global__ __launch_bounds__(kThreads * RS, (std::is_same<ET, float>::value ? 4 : 6)) void k_bmm_q(BmmArgs a)
{
    typedef BmOperand<P_CODED, P_TFAST, ET> OP;
    typedef BmOperand<!P_CODED, Q_TFAST, ET> OQ;
    typedef typename BmElem<false, ET>::global_t X;       // the plain operand's and the result's element type in memory
    constexpr bool kCut = std::is_same<ET, float>::value;
    constexpr int kTiles = (OP::kBytes + OQ::kBytes) * RS, kSums = RS > 1 ? 32 * kThreads * 4 : 0, kLds = kTiles > kSums ? kTiles : kSums;
    __shared__ __attribute__((aligned(16))) unsigned char lds_bm[kLds + (kCut ? 16 : 0)];
    int *large = reinterpret_cast<int *>(lds_bm + (kCut ? kLds : 0));   // binary32: some value is too large to be cut
    if (kCut && threadIdx.x == 0) *large = 0;

    const int group = RS > 1 ? __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kThreads) : 0;
    const int tid = RS > 1 ? int(threadIdx.x) % kThreads : int(threadIdx.x), lane = tid & 63, wave = tid >> 6;   // within the group
    unsigned char *LP = lds_bm + group * (OP::kBytes + OQ::kBytes), *LQ = LP + OP::kBytes;
    // grid: x = column tile, y = row tile, z = (sample, head) in pieces of at most 65535 (32-bit, uniform arithmetic only)
    const uint32_t b = blockIdx.z;
    const int r0 = int(blockIdx.y) * kBmTile, c0 = int(blockIdx.x) * kBmTile;
    const uint32_t h = (b + uint32_t(a.head0)) % uint32_t(a.heads);

    const X *xb = reinterpret_cast<const X *>(a.x) + int64_t(b) * a.x_batch + a.batch0 * a.x_batch;
    const int8_t *yb = a.y + int64_t(b) * a.y_batch + a.batch0 * a.y_batch;
    auto load_p = [&](int t0, int part) {
        if constexpr (P_CODED) return OP::load(yb, a.p_rs, a.p_ts, r0, t0, a.R, a.Tn, tid + part * kThreads);
        else return OP::load(xb, a.p_rs, a.p_ts, r0, t0, a.R, a.Tn, tid + part * kThreads);
    };
    auto load_q = [&](int t0, int part) {
        if constexpr (P_CODED) return OQ::load(xb, a.q_cs, a.q_ts, c0, t0, a.Cn, a.Tn, tid + part * kThreads);
        else return OQ::load(yb, a.q_cs, a.q_ts, c0, t0, a.Cn, a.Tn, tid + part * kThreads);
    };

    const int wr = wave >> 1, wc = wave & 1;            // 2 x 2 waves, a 32 x 32 MFMA tile each
    bm_v16f acc, acc1;
#pragma unroll
    for (int v = 0; v < 16; ++v) { acc[v] = 0.0f; acc1[v] = 0.0f; }
    bm_v8h ones;
#pragma unroll
    for (int j = 0; j < 8; ++j) ones[j] = __builtin_bit_cast(_Float16, BmNum<ET>::kOne);

    typename OP::Raw pv[kBmParts];
    typename OQ::Raw qv[kBmParts];
    float most = 0.0f;
#pragma unroll
    for (int k = 0; k < kBmParts; ++k) { pv[k] = load_p(group * kBmT, k); qv[k] = load_q(group * kBmT, k); }
    for (int first = 0; first < a.Tn; first += kBmT * RS) {   // the same count for every group: they meet at the barriers
        const int t0 = first + group * kBmT;
        __syncthreads();   // the previous stage's fragments have been read
#pragma unroll
        for (int k = 0; k < kBmParts; ++k) {
            OP::store(LP, pv[k], r0, t0, a.R, a.Tn, tid + k * kThreads);
            OQ::store(LQ, qv[k], c0, t0, a.Cn, a.Tn, tid + k * kThreads);
            if constexpr (kCut) {
                if constexpr (P_CODED) most = OQ::Elem::most(most, qv[k]);
                else most = OP::Elem::most(most, pv[k]);
            }
        }
        __syncthreads();
        if (first + kBmT * RS < a.Tn) {   // the next stage's loads fly while this one is multiplied
#pragma unroll
            for (int k = 0; k < kBmParts; ++k) { pv[k] = load_p(t0 + kBmT * RS, k); qv[k] = load_q(t0 + kBmT * RS, k); }
        }
#pragma unroll
        for (int ks = 0; ks < kBmT / 16; ++ks) {
            const bm_v8h coded = P_CODED ? OP::frag(LP, wr * 32, ks, lane) : OQ::frag(LQ, wc * 32, ks, lane);
            constexpr int kPlanes = OP::kPlanes * OQ::kPlanes;
#pragma unroll
            for (int q = kPlanes - 1; q >= 0; --q) {      // binary32: the smallest parts first
                const bm_v8h plain = P_CODED ? OQ::frag(LQ + q * OQ::kPlane, wc * 32, ks, lane) : OP::frag(LP + q * OP::kPlane, wr * 32, ks, lane);
                acc = BmNum<ET>::mfma(P_CODED ? coded : plain, P_CODED ? plain : coded, acc);
                acc1 = BmNum<ET>::mfma(P_CODED ? ones : plain, P_CODED ? plain : ones, acc1);
            }
        }
    }

    if constexpr (kCut) {
        if (too_large(most)) *large = 1;
        __syncthreads();
    }
    if constexpr (RS > 1) {
        float *sums = reinterpret_cast<float *>(lds_bm) + tid;
#pragma unroll 1
        for (int g = 1; g < RS; ++g) {
            __syncthreads();   // the last fragments, or the sums before, have been read
            if (group == g) {
#pragma unroll
                for (int v = 0; v < 16; ++v) { sums[v * kThreads] = acc[v]; sums[(16 + v) * kThreads] = acc1[v]; }
            }
            __syncthreads();
            if (group == 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) { acc[v] += sums[v * kThreads]; acc1[v] += sums[(16 + v) * kThreads]; }
            }
        }
        if (group != 0) return;
    }
    if constexpr (kCut) {
        if (*large) {                                     // uniform
            // the arguments are read again here, so that the ordinary path does not hold the strides to its end (it spilled for them)
            uint64_t args = reinterpret_cast<uint64_t>(__builtin_amdgcn_kernarg_segment_ptr());
            asm volatile("" : "+s"(args));
            bmm_plain_sums<P_CODED, float>(*reinterpret_cast<const BmmArgs *>(args), b, r0 + wr * 32 + (lane & 31), c0 + wc * 32 + (lane & 31), acc, acc1);
        } else {
#pragma unroll
            for (int v = 0; v < 16; ++v) { acc[v] *= kCutDown; acc1[v] *= kCutDown; }
        }
    }
    // lane l, register v of a 32 x 32 tile: row 8*(v/4) + 4*(l/32) + v%4, column l%32
    const float s = a.alpha[h] / 255.0f;
    const float off = fmaf(BmNum<ET>::kCentre, s, a.beta[h]);
    const int col = c0 + wc * 32 + (lane & 31);
    const int row_l = r0 + wr * 32 + (lane >> 5) * 4;
    // R * Cn < 2^31 (checked by the entry points): 32-bit offsets from the batch's base
    X *cb = reinterpret_cast<X *>(a.c) + (int64_t(b) + a.batch0) * a.c_batch;
    const uint32_t o0 = uint32_t(row_l) * uint32_t(a.Cn) + uint32_t(col);
    if (col < a.Cn) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int dr = (v >> 2) * 8 + (v & 3);
            if (row_l + dr < a.R) cb[o0 + uint32_t(dr) * uint32_t(a.Cn)] = BmNum<ET>::round(a.scale * fmaf(s, acc[v], off * acc1[v]));
        }
    }
}

template <bool P_CODED, bool P_TFAST, bool Q_TFAST, typename ET = _Float16>
static void launch_bmm(BmmArgs a, int64_t batches, hipStream_t s)
{
    a.tiles_r = int(ceil_div(a.R, kBmTile));
    a.tiles_c = int(ceil_div(a.Cn, kBmTile));
    // the z extent of a grid is limited to 65535: more (sample, head) pairs than that go in several launches
    for (int64_t b0 = 0; b0 < batches; b0 += 65535) {
        a.batch0 = b0;
        a.head0 = int(b0 % a.heads);
        const int64_t nb = batches - b0 < 65535 ? batches - b0 : 65535;
        const dim3 grid(unsigned(a.tiles_c), unsigned(a.tiles_r), unsigned(nb));
        const int64_t wgs = int64_t(a.tiles_c) * a.tiles_r * nb;
        // groups per workgroup: whole attention backward with 1 / 2 of them, by the workgroups of dV, dQ and dK: (4, 8, 577, 64), 320: 76 / 67 us;
        // (34, 4, 378, 64), 816: 93 / 102
        const int rs = a.Tn < 128 || wgs > 512 ? 1 : 2;
        if (rs == 2) hipLaunchKernelGGL((k_bmm_q<P_CODED, P_TFAST, Q_TFAST, ET, 2>), grid, dim3(kThreads * 2), 0, s, a);
        else hipLaunchKernelGGL((k_bmm_q<P_CODED, P_TFAST, Q_TFAST, ET, 1>), grid, dim3(kThreads), 0, s, a);
    }
}

// ---- few heads: a 32 x 32 tile per workgroup, its waves share out the contraction -----------------------------------
// The same product where all of it is a fraction of a round of workgroups, so that its time is latency: the stages of k_bmm_q, each
// with a trip to memory and two barriers, one after the other.  Here a wave takes every NW-th block of 16 contraction steps straight from
// memory (a lane: eight steps of one line -- a vector where they lie side by side, else eight loads that 32 lanes make whole
// lines of), all of them on their way at once, and the waves' tiles are added in LDS in a fixed order.  The sums of the
// plain operand are added by the lanes that hold it.  Same contracted values as k_bmm_q.  See bmm_waves for its range.
template <bool CODED, bool TFAST, typename ET> struct BmLane {
    typedef BmElem<CODED, ET> Elem;
    typedef typename Elem::global_t E;
    typedef typename std::conditional<sizeof(E) == 4, uint32_t, typename std::conditional<sizeof(E) == 2, uint16_t, uint8_t>::type>::type U;
    typename Elem::raw_t raw;

    // steps t .. t + 7 of the line; WHOLE: they all exist, else those from tn on read as zeros
    template <bool WHOLE> __device__ __forceinline__ void load(const E *base, int64_t line_stride, int64_t t_stride, int line, int t, int tn)
    {
        if (TFAST && WHOLE) {
            __builtin_memcpy(&raw, base + int64_t(line) * line_stride + t, 8 * sizeof(E));
            return;
        }
        const U *at = reinterpret_cast<const U *>(base) + int64_t(line) * (TFAST ? line_stride : 1);
        U e[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int tj = WHOLE || t + j < tn ? t + j : tn - 1;
            const U v = at[int64_t(tj) * (TFAST ? 1 : t_stride)];
            e[j] = WHOLE || t + j < tn ? v : U(0);
        }
        uint32_t w[sizeof(raw) / 4];
        constexpr int per = 4 / sizeof(E);
#pragma unroll
        for (int k = 0; k < int(sizeof(raw) / 4); ++k) {
            w[k] = uint32_t(e[per * k]);
#pragma unroll
            for (int j = 1; j < per; ++j) w[k] |= uint32_t(e[per * k + j]) << (32 / per * j);
        }
        __builtin_memcpy(&raw, w, sizeof(raw));
    }
};

template <typename ET, int NW> struct BmWavesLds {
    // sums of the plain operand's line lane % 32, this half's steps: the matrix cores added sixteen values with one rounding, eight binary32
    // values one by one do not (dA of 32-wide heads 6.3e-8 -> 6.9e-8), hence binary64
    typedef typename std::conditional<std::is_same<ET, float>::value, double, float>::type Sum;
    float sums[NW][16][64];                               // accumulator register v of a wave's lane
    Sum sums1[NW][64];
    int large[NW];                                        // the wave met a value that is too large to be cut
};

// what a product is: which operand is coded, and whose unit-stride index the contraction is
template <bool P_CODED_, bool P_TFAST_, bool Q_TFAST_> struct BmProduct {
    static constexpr bool P_CODED = P_CODED_, P_TFAST = P_TFAST_, Q_TFAST = Q_TFAST_;
};

template <typename PR, typename ET, int NW>
__device__ __forceinline__ void bmm_waves_tile(const BmmArgs &a, uint32_t block, BmWavesLds<ET, NW> &lds)
{
    constexpr bool P_CODED = PR::P_CODED, P_TFAST = PR::P_TFAST, Q_TFAST = PR::Q_TFAST;
    typedef typename BmElem<false, ET>::global_t X;
    typedef typename BmWavesLds<ET, NW>::Sum Sum;
    constexpr bool kCut = std::is_same<ET, float>::value;
    constexpr int kPlanes = BmElem<false, ET>::kPlanes;
    auto &sums = lds.sums;
    auto &sums1 = lds.sums1;
    auto &large = lds.large;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6), half = lane >> 5, l32 = lane & 31;
    const uint32_t tiles = uint32_t(a.tiles_r) * uint32_t(a.tiles_c);
    const uint32_t b = block / tiles, tile = block - b * tiles, tr = tile / uint32_t(a.tiles_c);
    const int r0 = int(tr) * 32, c0 = int(tile - tr * uint32_t(a.tiles_c)) * 32;
    const uint32_t h = b % uint32_t(a.heads);
    const X *xb = reinterpret_cast<const X *>(a.x) + int64_t(b) * a.x_batch;
    const int8_t *yb = a.y + int64_t(b) * a.y_batch;
    // lines beyond the extents are the last one again: they only reach results that are never written
    const int r = r0 + l32 < a.R ? r0 + l32 : a.R - 1, c = c0 + l32 < a.Cn ? c0 + l32 : a.Cn - 1;

    bm_v16f acc;
    Sum sum = 0;
    float most = 0.0f;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
    auto block16 = [&](int t0, auto whole) __attribute__((always_inline)) {
        constexpr bool WHOLE = decltype(whole)::value;
        BmLane<P_CODED, P_TFAST, ET> p;
        BmLane<!P_CODED, Q_TFAST, ET> q;
        if constexpr (P_CODED) {
            p.template load<WHOLE>(yb, a.p_rs, a.p_ts, r, t0 + half * 8, a.Tn);
            q.template load<WHOLE>(xb, a.q_cs, a.q_ts, c, t0 + half * 8, a.Tn);
        } else {
            p.template load<WHOLE>(xb, a.p_rs, a.p_ts, r, t0 + half * 8, a.Tn);
            q.template load<WHOLE>(yb, a.q_cs, a.q_ts, c, t0 + half * 8, a.Tn);
        }
        const auto &plain = [&]() -> const auto & { if constexpr (P_CODED) return q.raw; else return p.raw; }();
        const auto &code = [&]() -> const auto & { if constexpr (P_CODED) return p.raw; else return q.raw; }();
        const bm_v8h coded = BmNum<ET>::codes8(bm_v2i{int(code[0]), int(code[1])});
        u32x4 part[kPlanes];
        BmElem<false, ET>::cut(plain, part);
        if constexpr (kCut) {
            float x[8];
            __builtin_memcpy(x, &plain, 32);
#pragma unroll
            for (int j = 0; j < 8; ++j) sum += double(x[j]);
            most = BmElem<false, float>::most(most, plain);
        } else {
            const bm_v8h x = __builtin_bit_cast(bm_v8h, part[0]);
#pragma unroll
            for (int j = 0; j < 8; j += 2) sum = BmNum<ET>::dot_ones(x[j], x[j + 1], sum);
        }
#pragma unroll
        for (int k = kPlanes - 1; k >= 0; --k) {          // the smallest parts first
            const bm_v8h x = __builtin_bit_cast(bm_v8h, part[k]);
            acc = BmNum<ET>::mfma(P_CODED ? coded : x, P_CODED ? x : coded, acc);
        }
    };
    for (int t0 = wave * 16; t0 < a.Tn; t0 += NW * 16) {
        if (t0 + 16 <= a.Tn) block16(t0, std::true_type());
        else block16(t0, std::false_type());
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) sums[wave][v][lane] = acc[v];
    sums1[wave][lane] = sum;
    if constexpr (kCut) {
        const bool mine = __any(too_large(most));
        if (lane == 0) large[wave] = mine;
    }
    __syncthreads();
    float down = 1.0f;
    if constexpr (kCut) {
        down = kCutDown;
        if (__any(large[lane % NW])) {                    // the same in every wave: its steps again with binary32 products
            down = 1.0f;
            __syncthreads();
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
            for (int t0 = wave * 16; t0 < a.Tn; t0 += NW * 16)
                for (int t2 = t0; t2 < t0 + 16 && t2 < a.Tn; t2 += 2) {
                    const int t = t2 + half < a.Tn ? t2 + half : a.Tn - 1;
                    const int64_t po = int64_t(r) * a.p_rs + int64_t(t) * a.p_ts, qo = int64_t(t) * a.q_ts + int64_t(c) * a.q_cs;
                    const float code = float(int(yb[P_CODED ? po : qo])), x = t2 + half < a.Tn ? float(xb[P_CODED ? qo : po]) : 0.0f;
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(P_CODED ? code : x, P_CODED ? x : code, acc, 0, 0, 0);
                }
#pragma unroll
            for (int v = 0; v < 16; ++v) sums[wave][v][lane] = acc[v];
            __syncthreads();
        }
    }

    // a wave takes every NW-th register v of the tile: row 8 * (v / 4) + 4 * (lane / 32) + v % 4, column lane % 32
    const float s = a.alpha[h] / 255.0f, off = fmaf(BmNum<ET>::kCentre, s, a.beta[h]);
    X *cb = reinterpret_cast<X *>(a.c) + int64_t(b) * a.c_batch;
    const int col = c0 + l32;
    Sum of_col = 0;                                       // the sum of the plain operand's column
    if constexpr (P_CODED) {
#pragma unroll
        for (int w = 0; w < NW; ++w) of_col += sums1[w][l32] + sums1[w][32 + l32];
    }
#pragma unroll
    for (int v = wave; v < 16; v += NW) {
        const int rl = (v >> 2) * 8 + half * 4 + (v & 3);
        Sum t1 = of_col;
        if constexpr (!P_CODED) {                         // of its row: a part per lane of the half wave
            t1 = l32 < 2 * NW ? sums1[l32 / 2 % NW][(l32 & 1) * 32 + rl] : Sum(0);
#pragma unroll
            for (int x = 16; x > 0; x >>= 1) t1 += __shfl_xor(t1, x, 64);
        }
        float p[NW];
#pragma unroll
        for (int w = 0; w < NW; ++w) p[w] = sums[w][v][lane];
#pragma unroll
        for (int w = NW / 2; w > 0; w >>= 1)
#pragma unroll
            for (int i = 0; i < w; ++i) p[i] += p[i + w];
        if (r0 + rl < a.R && col < a.Cn)
            cb[uint32_t(r0 + rl) * uint32_t(a.Cn) + uint32_t(col)] = BmNum<ET>::round(a.scale * fmaf(s, p[0] * down, off * float(t1)));
    }
}

template <typename PR, typename ET, int NW>
__global__ __launch_bounds__(64 * NW) void k_bmm_waves(BmmArgs a)
{
    __shared__ BmWavesLds<ET, NW> lds;
    bmm_waves_tile<PR>(a, xcd_block(blockIdx.x, gridDim.x), lds);
}

// Two products of one call in one launch, the first one's tiles first: neither waits for the other, and a launch costs the host 3.7 us.
template <typename PR1, typename PR2, typename ET, int NW>
__global__ __launch_bounds__(64 * NW) void k_bmm_waves_two(BmmArgs a, BmmArgs b, uint32_t first)
{
    __shared__ BmWavesLds<ET, NW> lds;
    const uint32_t block = xcd_block(blockIdx.x, gridDim.x);
    if (block < first) bmm_waves_tile<PR1>(a, block, lds);   // uniform
    else bmm_waves_tile<PR2>(b, block - first, lds);
}

// Waves of k_bmm_waves's workgroups where it is the faster kernel for both products of a call, in one launch, else 0: no more than there are blocks of steps, and
// as many workgroups as run at once (binary32, whose other kernel is the general one alone: half as many again, or twice).  Two launches of the kernels chosen by
// da_way, tn_way and nn_way -> one of this kernel, dQ and dK: 16 bits (3, 436, 64) 14.0 -> 5.2, 400 to 512 tiles of eight waves -2.5, of four up to 450 -1.3 to -2, 512 to 610 -0.4 to +0.2, 720 +0.3 to +0.8; (1, 4096, 64) 96 -> 30,
// (2, 4100, 32) 91 -> 41, (4, 2048, 64) 54 -> 31, (1, 8192, 64) 185 -> 106.  binary32: (12, 783, 64), 600 tiles, 43 -> 32; (65, 112, 96), 780, 13.8 -> 10.9, (10, 1248, 64), 780, 47.0 -> 45.2.
// Four waves in binary32, heads of at most 32 columns, half a tile of the general kernel, (1653, 20, 32) 16.0 -> 12.5, (1951, 13, 32) 16.8 -> 13.7, (936, 35, 32), 1872, -0.4, others
// (290, 39, 64), 1160 tiles, 12.0 -> 10.6, (313, 22, 128), 1252, -0.1, (334, 57, 64), 1336, +0.5, (490, 53, 64), 1960, 12.8 -> 15.8, (464, 24, 128), 1856, 10.9 -> 14.4.
template <typename ET> static int bmm_waves(int64_t batches, int64_t R, int64_t Cn, int64_t Tn)
{
    constexpr bool kWide = std::is_same<ET, float>::value;
    const int64_t tiles = batches * ceil_div(R, 32) * ceil_div(Cn, 32);
    if (tiles <= 256 && Tn > 128) return 16;
    if (Tn > 64) return tiles <= (kWide ? 800 : 512) ? 8 : 0;
    return tiles <= (!kWide ? 640 : Cn <= 32 ? 2048 : 1248) ? 4 : 0;
}

// The same for a product in a launch of its own (dA or dV).  16 bits: four waves gain nothing there (dA +0.1 to +0.5 us, (78, 65, 64) 7.3 -> 8.5; dV -0.3 to +0.2), eight for dA
// -0.5 to 0 up to 512 tiles, but +0.5 from 257 on where two of them or fewer are one of the general kernel's and Dh has kernels of its own ((272, 27, 80) -0.6).  binary32: dA with four, 256 tiles -0.5, 512 0.0, 1024 +1.6, (490, 53, 64), 1960, +5.6 of 11.6, but -0.3 on average up to 2048 where a head is one tile; dV
// with four 1152 tiles -0.1, 1290 +1.0; with eight (65, 112, 96), 780, -0.6, long ones (2, 5311, 64), 664, -21 of 167, (6, 2047, 64), 768, -5 of 69,
// aligned (2, 5648, 64), 708, +5, (10, 1248, 64), 780, +6 of 43, but (3, 8192, 32), 768, -32.
template <typename ET> static int bmm_waves_alone(int64_t batches, int64_t R, int64_t Cn, int64_t Tn, bool da)
{
    constexpr bool kWide = std::is_same<ET, float>::value;
    const int nw = bmm_waves<ET>(batches, R, Cn, Tn);
    const int64_t tiles = batches * ceil_div(R, 32) * ceil_div(Cn, 32), general = batches * ceil_div(R, 64) * ceil_div(Cn, 64);
    if (nw == 4) return kWide && tiles <= (R <= 32 && Cn <= 32 ? 2048 : da ? 512 : 1248) ? 4 : 0;
    if (nw == 8 && kWide && Tn >= 1024 && Tn % 16 == 0 && Cn > 32 && tiles > 700) return 0;
    if (nw == 8 && !kWide && da && Tn % 32 == 0 && 2 * tiles < 5 * general && tiles > 256) return 0;
    return nw;
}

static int64_t bmm_waves_tiles(BmmArgs &a, int64_t batches)
{
    a.tiles_r = int(ceil_div(a.R, 32));
    a.tiles_c = int(ceil_div(a.Cn, 32));
    return batches * a.tiles_r * a.tiles_c;
}

template <bool P_CODED, bool P_TFAST, bool Q_TFAST, typename ET>
static bool launch_bmm_waves(BmmArgs a, int64_t batches, hipStream_t s)
{
    typedef BmProduct<P_CODED, P_TFAST, Q_TFAST> PR;
    const int nw = bmm_waves_alone<ET>(batches, a.R, a.Cn, a.Tn, P_TFAST && Q_TFAST);
    if (nw == 0) return false;
    const dim3 grid{unsigned(bmm_waves_tiles(a, batches))};
    if (nw == 16) hipLaunchKernelGGL((k_bmm_waves<PR, ET, 16>), grid, dim3(1024), 0, s, a);
    else if (nw == 8) hipLaunchKernelGGL((k_bmm_waves<PR, ET, 8>), grid, dim3(512), 0, s, a);
    else if constexpr (std::is_same<ET, float>::value) hipLaunchKernelGGL((k_bmm_waves<PR, ET, 4>), grid, dim3(256), 0, s, a);
    return true;
}

// Both products, where both of them would go that way; with different numbers of steps the shorter one's spare waves keep others from running,
// and two launches are the better ones from some 850 tiles on.  dA and dV / dQ and dK, two launches -> one: (6, 197, 64) f16 8.3 -> 5.0 / 9.1 -> 5.0 us, f32
// 9.0 -> 5.4 / 9.4 -> 5.2; (24, 97, 64) 7.3 -> 6.0 / 7.4 -> 5.0; dA and dV (12, 219, 64), 756 tiles, 8.9 -> 7.3, (16, 195, 64), 1008, 9.1 -> 8.4, (6, 330, 64) f32, 858, 10.3 -> 11.1,
// (9, 293, 64), 1080, 9.6 -> 10.2, (12, 398, 64) f32, 2340, 17 -> 26; dQ and dK (32, 248, 64), 1024, 10.5 -> 9.5.
template <typename PR1, typename PR2, typename ET>
static bool launch_bmm_waves_two(BmmArgs a, BmmArgs b, int64_t batches, hipStream_t s)
{
    const int na = bmm_waves<ET>(batches, a.R, a.Cn, a.Tn), nb = bmm_waves<ET>(batches, b.R, b.Cn, b.Tn);
    if (na == 0 || nb == 0) return false;
    const int64_t first = bmm_waves_tiles(a, batches), all = first + bmm_waves_tiles(b, batches);
    if (a.Tn != b.Tn && all > 850) return false;
    const int most = na > nb ? na : nb, nw = most == 16 && all > 256 ? 8 : most;
    const dim3 grid{unsigned(all)};
    if (nw == 16) hipLaunchKernelGGL((k_bmm_waves_two<PR1, PR2, ET, 16>), grid, dim3(1024), 0, s, a, b, uint32_t(first));
    else if (nw == 8) hipLaunchKernelGGL((k_bmm_waves_two<PR1, PR2, ET, 8>), grid, dim3(512), 0, s, a, b, uint32_t(first));
    else hipLaunchKernelGGL((k_bmm_waves_two<PR1, PR2, ET, 4>), grid, dim3(256), 0, s, a, b, uint32_t(first));
    return true;
}

template <typename PR1, typename PR2>
static bool launch_bmm_waves_two(BmmArgs a, BmmArgs b, int64_t batches, mesa_dtype dt, hipStream_t s)
{
    if (dt == MESA_F32) return launch_bmm_waves_two<PR1, PR2, float>(a, b, batches, s);
    if (dt == MESA_BF16) return launch_bmm_waves_two<PR1, PR2, __bf16>(a, b, batches, s);
    return launch_bmm_waves_two<PR1, PR2, _Float16>(a, b, batches, s);
}

// The plain kernel: bmm_plain_sums alone.  Kept simple: it serves extents shorter than one load vector.  T: the tensors'
// element type (BmmArgs' pointers are reinterpreted).
template <bool P_CODED, typename T>
__global__ __launch_bounds__(kThreads) void k_bmm_plain(BmmArgs a)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t b = blockIdx.z;
    const int r = int(blockIdx.y) * kBmTile + (wave >> 1) * 32 + (lane & 31);
    const int c = int(blockIdx.x) * kBmTile + (wave & 1) * 32 + (lane & 31);
    const uint32_t h = (b + uint32_t(a.head0)) % uint32_t(a.heads);
    const bool c_ok = c < a.Cn;
    bm_v16f acc, acc1;
    bmm_plain_sums<P_CODED, T>(a, b, r, c, acc, acc1);
    const float s = a.alpha[h] / 255.0f;
    const float off = fmaf(128.0f, s, a.beta[h]);
    const int row_l = int(blockIdx.y) * kBmTile + (wave >> 1) * 32 + (lane >> 5) * 4;
    const int64_t cb0 = (int64_t(b) + a.batch0) * a.c_batch;
    if (c_ok) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int rr = row_l + (v >> 2) * 8 + (v & 3);
            if (rr < a.R) Store<T>::store1(a.c, cb0 + int64_t(rr) * a.Cn + c, a.scale * fmaf(s, acc[v], off * acc1[v]));
        }
    }
}

template <bool P_CODED> static void launch_bmm_plain(BmmArgs a, int64_t batches, mesa_dtype dt, hipStream_t s)
{
    a.tiles_r = int(ceil_div(a.R, kBmTile));
    a.tiles_c = int(ceil_div(a.Cn, kBmTile));
    for (int64_t b0 = 0; b0 < batches; b0 += 65535) {
        a.batch0 = b0;
        a.head0 = int(b0 % a.heads);
        const int64_t nb = batches - b0 < 65535 ? batches - b0 : 65535;
#define MESA_LAUNCH_PLAIN(T) \
    hipLaunchKernelGGL((k_bmm_plain<P_CODED, T>), dim3(unsigned(a.tiles_c), unsigned(a.tiles_r), unsigned(nb)), dim3(kThreads), 0, s, a)
        MESA_FOR_DTYPE(dt, MESA_LAUNCH_PLAIN);
#undef MESA_LAUNCH_PLAIN
    }
}

// ---- the two products whose contraction index is the unit-stride index of BOTH operands' rows --------
// They need no transposition and (almost) no LDS: an MFMA operand fragment -- lane l: line l%32, the eight
// contraction slots 8*(l/32) ..+7 of a 16-slot step -- is one vector load straight from global memory.

// dA[i,j] = sum_d dO[i,d] * V_hat[j,d].  A workgroup takes 32 rows i of one head; its waves share out the
// blocks of 32 columns j.  Both operands' blocks are contiguous in memory (32 rows of dO, 32 rows of V
// codes): they come in as consecutive aligned 16-byte vectors -- a lane per row would cost the memory
// pipeline one access per lane -- and pass through LDS (dO once per workgroup, the codes privately per
// wave) into the fragments.  The MFMA runs with the operands exchanged (codes as the M side, dO as the N
// side), so that a lane ends up with ONE row i = l%32 and runs of four consecutive columns: the beta term's
// row sum of dO is then a per-lane scalar, and the tile goes to LDS with 8-byte writes.  The 32 x N output
// block is one contiguous piece of memory whose start is only element-aligned (N is odd for ViT): LDS holds
// it at the same offset from a 16-byte boundary, and it leaves as aligned 16-byte vectors; the few elements
// before the first and after the last whole vector are written one by one (the neighbouring blocks own the
// rest of those vectors).  Dh == 16 * KS, KS even.
// LDS: [output block, 64 N + 32 bytes | staged dO, 32 rows]  (the same space, one after the other in time),
// then 32 code rows per wave at `codes_at`.
// SOLO (short rows, N <= 64): a wave takes an item (head, block of 32 rows) all by itself, with its own
// piece of LDS and no barrier, so that no wave of the workgroup idles for want of column blocks.
template <int KS> struct DaCfg {
    static constexpr int Dh = 16 * KS;
    static constexpr int kRowO = 2 * Dh + 16;   // bytes per staged dO row (padded against bank conflicts)
    static constexpr int kRowV = Dh + 16;       // bytes per staged code row
    static constexpr int kVecO = Dh / 8;        // 16-byte vectors per dO row
    static constexpr int kVecV = Dh / 16;       // and per code row
    static constexpr int kCodeVecs = 32 * kVecV / 64;   // vectors per lane for a block of 32 code rows
    static constexpr int kWaves = kThreads / 64;
    // offset of the staged codes: behind the output block / the staged dO rows, whichever is longer
    static size_t codes_at(int64_t N)
    {
        const size_t out = size_t(N) * 64 + 32, stage = size_t(32) * kRowO;
        return ((out > stage ? out : stage) + 15) & ~size_t(15);
    }
    static size_t wave_bytes(int64_t N) { return codes_at(N) + size_t(32) * kRowV; }           // SOLO: per wave
    static size_t lds_bytes(int64_t N, bool solo) { return solo ? kWaves * wave_bytes(N) : codes_at(N) + size_t(kWaves) * 32 * kRowV; }
};

template <int KS, bool SOLO, typename ET>
__global__ __launch_bounds__(kThreads, KS <= 4 ? 7 : 4) void k_attn_da(const _Float16 *__restrict__ dO,
                                                                      const int8_t *__restrict__ vq, _Float16 *__restrict__ dA,
                                                                      int N, int heads, const float *__restrict__ alpha_v,
                                                                      const float *__restrict__ beta_v, int64_t batch0, int codes_at,
                                                                      unsigned items)
{
    typedef DaCfg<KS> C;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_all[];
    constexpr int Dh = C::Dh;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int fl = lane & 31, fk = (lane >> 5) * 8;
    const int nblocks = (N + 31) >> 5;
    // the threads that share an item, this thread's rank among them, and the column blocks this wave takes
    constexpr int kTeam = SOLO ? 64 : kThreads;
    const int t = SOLO ? lane : int(threadIdx.x);
    const int cb_first = SOLO ? 0 : wave, cb_step = SOLO ? 1 : C::kWaves;
    int64_t bh;
    int r0;
    if (SOLO) {                                            // items (at most 2^32) count (head, row block) pairs
        const unsigned item = blockIdx.x * C::kWaves + wave;
        if (item >= items) return;                         // no barrier in this mode
        const unsigned q = item / unsigned(nblocks);
        bh = q;
        r0 = int(item - q * unsigned(nblocks)) * 32;
    } else {
        bh = batch0 + blockIdx.y;
        r0 = int(blockIdx.x) * 32;
    }
    auto team_sync = [&]() {
        if constexpr (!SOLO) __syncthreads();
    };
    unsigned char *lds_da = SOLO ? lds_all + wave * (codes_at + 32 * C::kRowV) : lds_all;
    unsigned char *lv = SOLO ? lds_da + codes_at : lds_all + codes_at + wave * (32 * C::kRowV);
    constexpr int kOVecs = (32 * C::kVecO + kTeam - 1) / kTeam;   // dO vectors per thread
    const int code_vecs = N * C::kVecV;                    // of one head
    const int rows = N - r0 < 32 ? N - r0 : 32;
    const u32x4 *vvec = reinterpret_cast<const u32x4 *>(vq + bh * N * int64_t(Dh));
    auto load_codes = [&](int c0, u32x4 (&raw)[C::kCodeVecs]) {
#pragma unroll
        for (int i = 0; i < C::kCodeVecs; ++i) {
            const int g = c0 * C::kVecV + lane + 64 * i;   // rows past the head's end repeat its last vector; never used
            raw[i] = vvec[g < code_vecs ? g : code_vecs - 1];
        }
    };
    auto store_codes = [&](const u32x4 (&raw)[C::kCodeVecs]) {
#pragma unroll
        for (int i = 0; i < C::kCodeVecs; ++i) {
            const int idx = lane + 64 * i;
            *reinterpret_cast<u32x4 *>(lv + (idx / C::kVecV) * C::kRowV + (idx % C::kVecV) * 16) = raw[i];
        }
    };
    u32x4 raw[C::kCodeVecs];
    if (cb_first < nblocks) load_codes(cb_first * 32, raw);
    {
        const int o_vecs = rows * C::kVecO;
        const u32x4 *ovec = reinterpret_cast<const u32x4 *>(dO + (bh * N + r0) * int64_t(Dh));
        u32x4 ov[kOVecs];
#pragma unroll
        for (int k = 0; k < kOVecs; ++k) {                 // rows past the last one repeat its last vector
            const int idx = t + k * kTeam;
            ov[k] = ovec[idx < o_vecs ? idx : o_vecs - 1];
        }
#pragma unroll
        for (int k = 0; k < kOVecs; ++k) {
            const int idx = t + k * kTeam;
            if (idx < 32 * C::kVecO) *reinterpret_cast<u32x4 *>(lds_da + (idx / C::kVecO) * C::kRowO + (idx % C::kVecO) * 16) = ov[k];
        }
    }
    team_sync();
    bm_v8h fo[KS];
    float rsum = 0.0f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        fo[ks] = *reinterpret_cast<const bm_v8h *>(lds_da + fl * C::kRowO + (ks * 16 + fk) * 2);
#pragma unroll
        for (int j = 0; j < 8; j += 2)
            rsum = BmNum<ET>::dot_ones(fo[ks][j], fo[ks][j + 1], rsum);
    }
    rsum += __shfl_xor(rsum, 32);                          // both halves of the row's slots
    team_sync();                                           // every wave holds its fragments: the space becomes the output block
    const int h = int(bh % heads);
    const float s = alpha_v[h] / 255.0f;
    const float add = fmaf(BmNum<ET>::kCentre, s, beta_v[h]) * rsum;

    const int64_t e0 = (bh * N + r0) * int64_t(N);         // first element of the output block
    const int mis = int(e0 & 7);                           // its offset from a 16-byte boundary, in elements
    _Float16 *lo = reinterpret_cast<_Float16 *>(lds_da);    // element (i, j) of the block at mis + i * N + j

    for (int cbk = cb_first; cbk < nblocks; cbk += cb_step) {
        const int c0 = cbk * 32;
        store_codes(raw);
        if (cbk + cb_step < nblocks) load_codes(c0 + 32 * cb_step, raw);   // the wave's next block
        bm_v8h fc[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) fc[ks] = BmNum<ET>::codes8(*reinterpret_cast<const bm_v2i *>(lv + fl * C::kRowV + ks * 16 + fk));
        bm_v16f acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) acc = BmNum<ET>::mfma(fc[ks], fo[ks], acc);
        // lane l, register v: column c0 + 8*(v/4) + 4*(l/32) + v%4, row l%32
        if (fl < rows) {
            const int at = mis + fl * N + c0 + (lane >> 5) * 4;
            if (c0 + 32 <= N) {                            // uniform: the whole column block lies inside
                // Four consecutive elements from an element-aligned position, with aligned writes only
                // (LDS stalls for dozens of cycles on a misaligned 8-byte write): the first and the last
                // element alone, the 4-byte word that holds elements 1, 2 (odd position) or 0, 1 (even),
                // and element 2 (even) or, again, 3 (odd).
                const bool odd = at & 1;
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    bm_v4h o;
#pragma unroll
                    for (int k = 0; k < 4; ++k) o[k] = BmNum<ET>::round(fmaf(s, acc[4 * g + k], add));
                    _Float16 *q = lo + at + 8 * g;
                    q[0] = o[0];
                    q[3] = o[3];
                    *reinterpret_cast<bm_v2h *>(q + (odd ? 1 : 0)) = odd ? bm_v2h{o[1], o[2]} : bm_v2h{o[0], o[1]};
                    q[odd ? 3 : 2] = odd ? o[3] : o[2];
                }
            } else {
#pragma unroll
                for (int g = 0; g < 4; ++g)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (c0 + (lane >> 5) * 4 + 8 * g + k < N) lo[at + 8 * g + k] = BmNum<ET>::round(fmaf(s, acc[4 * g + k], add));
            }
        }
    }
    team_sync();

    // the block leaves: elements [e0, e1) of dA; LDS element x holds global element (e0 - mis) + x
    const int total = rows * N;
    const int64_t ebase = e0 - mis;
    const int v_first = (mis + 7) >> 3, v_end = (mis + total) >> 3;   // whole vectors, in units of 8 elements from ebase
    for (int v = v_first + t; v < v_end; v += kTeam)
        *reinterpret_cast<u32x4 *>(dA + ebase + 8 * int64_t(v)) = *reinterpret_cast<const u32x4 *>(lo + 8 * v);
    if (t < 8) {                                            // before the first whole vector
        const int x = mis + t;
        if (x < 8 * v_first && x < mis + total) dA[ebase + x] = lo[x];
    } else if (t < 16) {                                    // after the last one
        const int x = 8 * v_end + (t - 8);
        if (x >= 8 * v_first && x < mis + total) dA[ebase + x] = lo[x];
    }
}

// ---- dA by tiles of columns (long sequences, and aligned ones) ----------
// A workgroup takes 64 rows i and 256 columns j of one head: the 64 rows of dO and the 256 rows of V codes go to LDS
// once (the codes only until every wave holds its fragments), wave w multiplies the 64 rows by the code rows 64 w ..+63 (four accumulator tiles, codes on the M side as in
// k_attn_da: a lane ends up with one row i and runs of four consecutive j), and its 64 x 64 piece of the result leaves
// through a private LDS region, 32 rows at a time, as aligned 16-byte vectors: 128 contiguous bytes per row and wave,
// 512 per row and workgroup.  The column tiles of a row block are neighbours, on one XCD.  Rows that start at any element (ANY) leave by
// unaligned stores, the last few elements of a row one by one.  Dh == 16 * KS.
template <int KS> struct DcCfg {
    static constexpr int Dh = 16 * KS;
    static constexpr int kRowO = 2 * Dh + 16, kRowV = Dh + 16;     // bytes per staged row of dO, of codes
    static constexpr int kRowOut = 64 * 2 + 16;                    // bytes per staged row of a wave's result
    static constexpr int kVecO = Dh / 8, kVecV = Dh / 16;
    // the waves' result regions take the place of the codes once every wave holds its code fragments
    static constexpr int kRows = KS <= 4 ? 128 : 64;               // rows of dO per workgroup (the codes are read once for all of them)
    static constexpr int kCodesAt = kRows * kRowO, kOutAt = kCodesAt;
    static constexpr int kLds = kCodesAt + (256 * kRowV > 4 * 32 * kRowOut ? 256 * kRowV : 4 * 32 * kRowOut);
};

template <int KS, bool ANY, typename ET>
__global__ __launch_bounds__(kThreads, KS <= 4 ? 3 : 2) void k_attn_da_cols(const _Float16 *__restrict__ dO, const int8_t *__restrict__ vq,
                                                                            _Float16 *__restrict__ dA, int N, int heads, int tiles_j,
                                                                            int tiles_i, int on_lines, const float *__restrict__ alpha_v,
                                                                            const float *__restrict__ beta_v)
{
    typedef DcCfg<KS> C;
    __shared__ __attribute__((aligned(16))) unsigned char lds_dc[C::kLds];
    constexpr int Dh = C::Dh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int fl = lane & 31, fk = (lane >> 5) * 8;
    const unsigned bid = xcd_block(blockIdx.x, gridDim.x);
    const unsigned tj = bid % unsigned(tiles_j), rest = bid / unsigned(tiles_j);
    const int64_t bh = rest / unsigned(tiles_i);
    const int i0 = int(rest % unsigned(tiles_i)) * C::kRows, j0 = int(tj) * 256;
    const int rows = N - i0 < C::kRows ? N - i0 : C::kRows, cols = N - j0 < 256 ? N - j0 : 256;

    {   // staging: rows past the end repeat the last one (their results are never written)
        const u32x4 *ovec = reinterpret_cast<const u32x4 *>(dO + (bh * N + i0) * int64_t(Dh));
        const int o_vecs = rows * C::kVecO;
#pragma unroll
        for (int k = 0; k < (C::kRows * C::kVecO + kThreads - 1) / kThreads; ++k) {
            const int idx = tid + k * kThreads;
            if (idx < C::kRows * C::kVecO)
                *reinterpret_cast<u32x4 *>(lds_dc + (idx / C::kVecO) * C::kRowO + (idx % C::kVecO) * 16) = ovec[idx < o_vecs ? idx : o_vecs - 1];
        }
        const u32x4 *vvec = reinterpret_cast<const u32x4 *>(vq + (bh * N + j0) * int64_t(Dh));
        const int v_vecs = cols * C::kVecV;
#pragma unroll
        for (int k = 0; k < 256 * C::kVecV / kThreads; ++k) {
            const int idx = tid + k * kThreads;
            *reinterpret_cast<u32x4 *>(lds_dc + C::kCodesAt + (idx / C::kVecV) * C::kRowV + (idx % C::kVecV) * 16) = vvec[idx < v_vecs ? idx : v_vecs - 1];
        }
    }
    __syncthreads();
    const int h = int(bh % heads);
    const float s = alpha_v[h] / 255.0f;
    const float off = fmaf(BmNum<ET>::kCentre, s, beta_v[h]);
    unsigned char *lout = lds_dc + C::kOutAt + wave * (32 * C::kRowOut);
    // on_lines (da_streams): the pieces of a row are whole lines, or halves of one, that nobody of this launch reads, and leave non-temporally
    const Span lines(dA + (bh * N + i0) * int64_t(N), uint32_t(rows) * uint32_t(N) * 2u);
    auto wave_sync = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    // the codes of this wave's 64 columns, as operands: lane l holds code row l%32 (+32), slots 8*(l/32) ..+7 of a step
    bm_v8h fc[2][KS];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            fc[jb][ks] = BmNum<ET>::codes8(*reinterpret_cast<const bm_v2i *>(lds_dc + C::kCodesAt + (wave * 64 + jb * 32 + fl) * C::kRowV + ks * 16 + fk));
    __syncthreads();                                       // the codes' place becomes the result regions
    if (wave * 64 >= cols) return;                         // this wave's columns lie past N (no barrier follows)
#pragma unroll
    for (int rb = 0; rb < C::kRows / 32; ++rb) {
        if (rb * 32 >= rows) break;                        // uniform
        bm_v8h fo[KS];
        float rsum = 0.0f;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            fo[ks] = *reinterpret_cast<const bm_v8h *>(lds_dc + (rb * 32 + fl) * C::kRowO + (ks * 16 + fk) * 2);
#pragma unroll
            for (int j = 0; j < 8; j += 2) rsum = BmNum<ET>::dot_ones(fo[ks][j], fo[ks][j + 1], rsum);
        }
        rsum += __shfl_xor(rsum, 32);                      // both halves of the row's slots
        const float add = off * rsum;
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) {
            bm_v16f acc;
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) acc = BmNum<ET>::mfma(fc[jb][ks], fo[ks], acc);
            // lane l, register v: column 32*jb + 8*(v/4) + 4*(l/32) + v%4 of the wave's 64, row l%32
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                bm_v4h o;
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k] = BmNum<ET>::round(fmaf(s, acc[4 * g + k], add));
                *reinterpret_cast<bm_v4h *>(lout + fl * C::kRowOut + (jb * 32 + 8 * g + (lane >> 5) * 4) * 2) = o;
            }
        }
        wave_sync();
        // 32 rows x eight vectors of eight columns: lane l takes vector l%8 of rows l/8, l/8 + 8, ..
        const int cv = lane & 7;
        if (wave * 64 + cv * 8 < cols) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int r = (lane >> 3) + 8 * k;
                if (rb * 32 + r < rows) {
                    _Float16 *to = dA + (bh * N + i0 + rb * 32 + r) * int64_t(N) + j0 + wave * 64 + cv * 8;
                    const u32x4 w = *reinterpret_cast<const u32x4 *>(lout + r * C::kRowOut + cv * 16);
                    if constexpr (!ANY) {
                        if (on_lines) lines.store16(uint32_t((rb * 32 + r) * N + j0 + wave * 64 + cv * 8) * 2u, w);
                        else *reinterpret_cast<u32x4 *>(to) = w;
                    } else if (wave * 64 + cv * 8 + 8 <= cols) {
                        __builtin_memcpy(to, &w, 16);      // rows start at any element
                    } else {
                        _Float16 e[8];
                        __builtin_memcpy(e, &w, 16);
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            if (wave * 64 + cv * 8 + q < cols) to[q] = e[q];
                    }
                }
            }
        }
        wave_sync();                                       // the region is free for the next 32 rows
    }
}

// ---- the two products that contract over the ROW index of both operands: dK = scale * dS^T Q_hat, dV = A_hat^T dO ----
// One workgroup per head.  It walks down the rows i in chunks of 32: the chunk of the N x N operand (dS or the
// A codes) is one contiguous, merely element-aligned piece of memory that comes in as aligned 16-byte
// vectors and lies in LDS as it lies in memory; the chunk of the N x Dh operand (Q codes or dO) has aligned
// rows and goes to LDS row by row.  The next chunk's loads are in flight while a chunk is multiplied
// (two LDS buffers, one barrier per chunk).  The waves share out the blocks of 32 output rows j.  An MFMA
// fragment of the N x N operand -- lane l: column j = l%32, the eight rows 8*(l/32) ..+7 of a 16-row step --
// is gathered from LDS with eight 2-byte (1-byte) reads a row apart; the fragment of the other operand comes
// from transposing reads.  The MFMA runs with the N x Dh operand on the M side, so a lane ends up with one
// output row j and runs of four consecutive d.  Dh == 32 * DT; N <= 32 * NW (a block of j per wave): below 128, longer heads go by tiles (tn_way).
template <int DT, bool WIDE_CODED, int NW> struct TnCfg {
    static constexpr int kNt = 64 * NW;                     // threads of a workgroup (NW waves)
    // WIDE_CODED: the N x N operand is the coded one (dV: A codes, dO plain); else dK: dS plain, Q codes
    static constexpr int Dh = 32 * DT;
    static constexpr int kWideEb = WIDE_CODED ? 1 : 2;     // bytes per element of the N x N operand
    static constexpr int kRowNarrow = WIDE_CODED ? 2 * Dh + 32 : Dh + 32;   // bytes per staged row of the N x Dh operand
    static constexpr int kNarrowVecs = 32 * Dh * (WIDE_CODED ? 2 : 1) / 16;   // 16-byte vectors per chunk of it
    static constexpr int kMaxWideVecs = 4;                 // vectors of the N x N chunk per thread kept in flight
    static size_t wide_bytes(int64_t N) { return (size_t(32) * N * kWideEb + 16 + 64 + 15) & ~size_t(15); }
    static size_t narrow_bytes() { return size_t(32) * kRowNarrow; }
    static size_t lds_bytes(int64_t N) { return 2 * (wide_bytes(N) + narrow_bytes()); }
};

// waves per SIMD the register budget is set for (the accumulators are 16 * DT registers)
template <int DT, int NW> constexpr int tn_waves_per_simd() { return (NW < 4 ? DT <= 2 : DT < 4) ? 3 : 2; }

template <int DT, bool WIDE_CODED, int NW, typename ET>
__global__ __launch_bounds__(64 * NW, (tn_waves_per_simd<DT, NW>())) void k_attn_tn(const void *__restrict__ wide_, const void *__restrict__ narrow_,
                                                         _Float16 *__restrict__ out, int N, int heads, float scale,
                                                         const float *__restrict__ alpha, const float *__restrict__ beta,
                                                         int wide_bytes, int64_t wide_elems)
{
    typedef TnCfg<DT, WIDE_CODED, NW> C;
    constexpr int kNt = C::kNt;
    typedef typename BmElem<WIDE_CODED, ET>::global_t WideT;       // element of the N x N operand
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_tn[];
    constexpr int Dh = C::Dh;
    constexpr int kEw = 16 / C::kWideEb;                   // elements of the N x N operand per 16-byte vector
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t bh = blockIdx.x;
    const WideT *wide = static_cast<const WideT *>(wide_);
    const unsigned char *narrow = static_cast<const unsigned char *>(narrow_) + bh * N * int64_t(Dh) * (WIDE_CODED ? 2 : 1);
    const int fl = lane & 31, half = lane >> 5;
    const int nchunks = (N + 31) >> 5;
    // LDS: [chunk of the N x N operand] x 2, then [chunk of the N x Dh operand] x 2 (offsets, so that the
    // accesses stay LDS accesses)
    auto buf_w = [&](int b) { return lds_tn + b * wide_bytes; };
    auto buf_n = [&](int b) { return lds_tn + 2 * wide_bytes + b * (32 * C::kRowNarrow); };

    // ---- staging -------------------------------------------------------------------------------------
    u32x4 wv[C::kMaxWideVecs], nv[(C::kNarrowVecs + kNt - 1) / kNt];
    int mis = 0, nvec = 0, whole = 0;                      // of the chunk held in wv
    auto chunk_geom = [&](int c, int &mis_, int &nvec_, int &whole_, int64_t &ebase_) {
        const int i0 = c * 32;
        const int rows = N - i0 < 32 ? N - i0 : 32;
        const int64_t e0 = (bh * N + i0) * int64_t(N);     // first element of the chunk
        mis_ = int(e0 & (kEw - 1));
        ebase_ = e0 - mis_;
        nvec_ = (mis_ + rows * N + kEw - 1) / kEw;
        // the last vector of the whole tensor may reach past its end: that one is read element by element
        whole_ = wide_elems - ebase_ >= int64_t(nvec_) * kEw ? nvec_ : nvec_ - 1;
    };
    auto load_chunk = [&](int c) {
        int64_t ebase;
        chunk_geom(c, mis, nvec, whole, ebase);
        const u32x4 *src = reinterpret_cast<const u32x4 *>(wide + ebase);
#pragma unroll
        for (int k = 0; k < C::kMaxWideVecs; ++k) {
            const int v = tid + k * kNt;
            if (v < whole) wv[k] = src[v];
        }
        const u32x4 *nsrc = reinterpret_cast<const u32x4 *>(narrow + int64_t(c) * 32 * Dh * (WIDE_CODED ? 2 : 1));
        const int nrows = N - c * 32 < 32 ? N - c * 32 : 32;
        const int nvecs = nrows * (C::kNarrowVecs / 32);
#pragma unroll
        for (int k = 0; k < int(sizeof(nv) / sizeof(nv[0])); ++k) {
            const int v = tid + k * kNt;
            if (v < nvecs) nv[k] = nsrc[v];
            else nv[k] = u32x4{0u, 0u, 0u, 0u};            // rows past the end: zeros (codes of 0 / plain zeros)
        }
    };
    auto store_chunk = [&](int c, int b) {
        unsigned char *lw = buf_w(b);
#pragma unroll
        for (int k = 0; k < C::kMaxWideVecs; ++k) {
            const int v = tid + k * kNt;
            if (v < whole) *reinterpret_cast<u32x4 *>(lw + v * 16) = wv[k];
        }
        if (whole < nvec && tid < kEw) {                   // the tensor's very last, partial vector
            int64_t ebase;
            int m_, n_, w_;
            chunk_geom(c, m_, n_, w_, ebase);
            const int64_t g = ebase + int64_t(whole) * kEw + tid;
            reinterpret_cast<WideT *>(lw)[whole * kEw + tid] = g < wide_elems ? wide[g] : WideT(0);
        }
        constexpr int kVecRow = C::kNarrowVecs / 32;
#pragma unroll
        for (int k = 0; k < int(sizeof(nv) / sizeof(nv[0])); ++k) {
            const int v = tid + k * kNt;
            if (v < C::kNarrowVecs) *reinterpret_cast<u32x4 *>(buf_n(b) + (v / kVecRow) * C::kRowNarrow + (v % kVecRow) * 16) = nv[k];
        }
    };

    // ---- accumulators: wave w takes the block j = 32 * w ----------------------------------
    const int j0 = wave * 32;
    bm_v16f acc[DT];
    bm_v16f acc1[WIDE_CODED ? DT : 1];                     // dV: column sums of dO per d, from MFMAs against ones
    float csum = 0.0f;                                     // dK: column sums of dS per j, per lane
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[dt][v] = 0.0f;
#pragma unroll
    for (int dt = 0; dt < (WIDE_CODED ? DT : 1); ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc1[dt][v] = 0.0f;
    bm_v8h ones;
#pragma unroll
    for (int j = 0; j < 8; ++j) ones[j] = __builtin_bit_cast(_Float16, BmNum<ET>::kOne);
    const int blk = lane >> 4, sl = lane & 15;

    load_chunk(0);
    for (int c = 0; c < nchunks; ++c) {
        const int b = c & 1;
        const int mis_c = mis;
        store_chunk(c, b);
        if (c + 1 < nchunks) load_chunk(c + 1);
        __syncthreads();   // chunk c is in LDS; every wave has finished with chunk c - 1 (the other buffer)
        const int rows = N - c * 32 < 32 ? N - c * 32 : 32;
        const WideT *lw = reinterpret_cast<const WideT *>(buf_w(b));
        const unsigned char *ln = buf_n(b);
        const bool ragged = rows < 32;                     // uniform: the head's last chunk
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            if (ks * 16 >= rows) break;                    // uniform
            // fragments of the N x Dh operand: lane: d = 32*dt + l%32, rows 16*ks + 8*(l/32) ..+7
            bm_v8h fn[DT];
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                if (WIDE_CODED) {
                    const unsigned char *p = ln + (ks * 16 + (blk >> 1) * 8 + (sl >> 2)) * C::kRowNarrow + (dt * 32 + (blk & 1) * 16 + (sl & 3) * 4) * 2;
                    const bm_v4h lo = __builtin_bit_cast(bm_v4h, __builtin_amdgcn_ds_read_tr16_b64_v4i16(BM_LDS3(bm_v4s, p)));
                    const bm_v4h hi = __builtin_bit_cast(bm_v4h, __builtin_amdgcn_ds_read_tr16_b64_v4i16(BM_LDS3(bm_v4s, p + 4 * C::kRowNarrow)));
                    fn[dt] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                    acc1[dt] = BmNum<ET>::mfma(fn[dt], ones, acc1[dt]);
                } else {
                    const unsigned char *p = ln + (ks * 16 + (blk >> 1) * 8 + (sl >> 1)) * C::kRowNarrow + dt * 32 + (blk & 1) * 16 + (sl & 1) * 8;
                    fn[dt] = BmNum<ET>::codes8(__builtin_amdgcn_ds_read_tr8_b64_v2i32(BM_LDS3(bm_v2i, p)));
                }
            }
            if (j0 < N) {                                  // uniform per wave
                const int j = j0 + fl < N ? j0 + fl : N - 1;   // columns past the end repeat the last one; never written
                const int at = mis_c + (ks * 16 + half * 8) * N + j;
                bm_v8h fw;
                if (WIDE_CODED) {
                    // rows past the end meet zeros of the other operand: any code will do there
                    bm_v4u u;
#pragma unroll
                    for (int k = 0; k < 4; ++k)            // two codes per register: bits 0-7 and 16-23
                        u[k] = unsigned(reinterpret_cast<const unsigned char *>(lw)[at + (2 * k) * N]) |
                               (unsigned(reinterpret_cast<const unsigned char *>(lw)[at + (2 * k + 1) * N]) << 16);
                    fw = BmNum<ET>::gathered(u);           // stored bytes -> operand values
                } else {
#pragma unroll
                    for (int k = 0; k < 8; ++k) fw[k] = reinterpret_cast<const _Float16 *>(lw)[at + k * N];
                    if (ragged) {                          // rows past the end: zeros (LDS holds stale data there)
                        bm_v4u w4 = __builtin_bit_cast(bm_v4u, fw);
                        const int r = ks * 16 + half * 8;
#pragma unroll
                        for (int k = 0; k < 4; ++k) w4[k] &= (r + 2 * k < rows ? 0xffffu : 0u) | (r + 2 * k + 1 < rows ? 0xffff0000u : 0u);
                        fw = __builtin_bit_cast(bm_v8h, w4);
                    }
#pragma unroll
                    for (int k = 0; k < 8; k += 2)
                        csum = BmNum<ET>::dot_ones(fw[k], fw[k + 1], csum);
                }
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) acc[dt] = BmNum<ET>::mfma(fn[dt], fw, acc[dt]);
            }
        }
    }

    // ---- epilogue: lane l, register v of a tile: d = 32*dt + 8*(v/4) + 4*(l/32) + v%4, row j = j0 + l%32 ----
    const int h = int(bh % heads);
    const float s = alpha[h] / 255.0f;
    const float off = fmaf(BmNum<ET>::kCentre, s, beta[h]);
    const int j = j0 + fl;
    if (j >= N) return;
    float cs = 0.0f;
    if (!WIDE_CODED) cs = off * (csum + __shfl_xor(csum, 32));
    _Float16 *po = out + (bh * N + j) * int64_t(Dh) + half * 4;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bm_v4h o;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float add = WIDE_CODED ? off * acc1[dt][4 * g + k] : cs;
                o[k] = BmNum<ET>::round(scale * fmaf(s, acc[dt][4 * g + k], add));
            }
            *reinterpret_cast<bm_v4h *>(po + dt * 32 + g * 8) = o;
        }
}

// ---- the same two products by tiles of columns -----
// A workgroup takes 256 columns j of one head and walks down ALL rows i in chunks of 16: per chunk 16 row segments of
// 256 elements of the N x N operand (512 contiguous bytes of dS, 256 of the A codes: 16-byte vectors, aligned where N is
// a multiple of 16) and the chunk's 16 rows of the N x Dh operand.  Both lie in LDS row by row, with a
// pitch that keeps the transposing reads of sixteen lanes on different banks; every MFMA operand is one or two
// transposing reads (lane: column j or d, eight consecutive rows i).  The next chunk's vectors wait in registers
// while a chunk is multiplied (two LDS buffers, one barrier per chunk).  Wave w takes columns 64 w ..+63 of the tile.
// The workgroups of a head's column tiles are neighbours on one XCD: they read adjacent segments of the same rows at
// about the same time and share the N x Dh chunks in the L2 (dealt out over the XCDs: 3 to 9 % slower, with the other two kernels of its kind).  The N x N operand is read exactly once.
// As in k_attn_tn the N x Dh operand sits on the M side: a lane ends up with one output row j and runs of four d.
//
// RS: groups of four waves that share out the workgroup's chunks (group g takes chunks g, g + RS, ...), each with LDS buffers
// of its own; their sums are added through LDS at the end, in group order.  Few heads leave a CU one or two workgroups,
// and one workgroup of four waves has a single chunk of 4 to 8 KB on its way: latency, not HBM, is what it waits for.
template <int DT, bool WIDE_CODED, int RS> struct TcCfg {
    static constexpr int Dh = 32 * DT;
    static constexpr int kJW = 256;                        // columns of the N x N operand per workgroup
    static constexpr int kNt = kJW;                        // threads of a group: a wave per 64 columns (two blocks of 32)
    static constexpr int kJB = 2;
    static constexpr int kCR = 16;                         // rows per chunk
    static constexpr int kAhead = WIDE_CODED ? 2 : 1;      // chunks in registers ahead of the one in LDS: the codes' chunks are
                                                           // half the bytes, and it is bytes in flight that hide the latency
    static constexpr int kWideEb = WIDE_CODED ? 1 : 2;
    static constexpr int kPitchW = kJW * kWideEb + (WIDE_CODED ? 16 : 32);   // bytes per staged row segment
    static constexpr int kVecRowW = kJW * kWideEb / 16;    // 16-byte vectors per row segment
    static constexpr int kWideVecs = kCR * kVecRowW / kNt;   // per thread and chunk: 4 (binary16) or 2 (codes)
    static constexpr int kRowN = WIDE_CODED ? 2 * Dh + 32 : Dh + 32;   // bytes per staged row of the N x Dh operand
    static constexpr int kVecRowN = Dh * (WIDE_CODED ? 2 : 1) / 16;
    static constexpr int kNarrowVecs = (kCR * kVecRowN + kNt - 1) / kNt;
    static constexpr int kStage = kCR * kPitchW + kCR * kRowN;
    static constexpr int kSum = (kJB * DT * 16 + kJB + DT) * kNt * 4;   // a group's sums
    static constexpr int kLds = RS * 2 * kStage > (RS > 1 ? kSum : 0) ? RS * 2 * kStage : kSum;
    static constexpr int kWaves = RS > 1 ? RS : 2;         // per SIMD, for the register budget
};

template <int DT, bool WIDE_CODED, int RS, bool ANY, typename ET>
__global__ __launch_bounds__((TcCfg<DT, WIDE_CODED, RS>::kNt * RS), (TcCfg<DT, WIDE_CODED, RS>::kWaves)) void k_attn_tn_cols(const void *__restrict__ wide_, const void *__restrict__ narrow_,
                                                              _Float16 *__restrict__ out, int N, int heads, int tiles_j, float scale,
                                                              const float *__restrict__ alpha, const float *__restrict__ beta)
{
    typedef TcCfg<DT, WIDE_CODED, RS> C;
    __shared__ __attribute__((aligned(16))) unsigned char lds_all[C::kLds];
    constexpr int Dh = C::Dh;
    const int group = RS > 1 ? __builtin_amdgcn_readfirstlane(int(threadIdx.x) / C::kNt) : 0;
    const int tid = RS > 1 ? int(threadIdx.x) % C::kNt : int(threadIdx.x);   // within the group
    const int lane = tid & 63, wave = tid >> 6;
    unsigned char *lds_tc = lds_all + group * 2 * C::kStage;
    const unsigned bid = xcd_block(blockIdx.x, gridDim.x);
    const int64_t bh = bid / unsigned(tiles_j);
    const int j0 = int(bid % unsigned(tiles_j)) * C::kJW;
    const bool last_head = ANY && bid + unsigned(tiles_j) >= gridDim.x;
    const unsigned char *wide = static_cast<const unsigned char *>(wide_) + (bh * N * int64_t(N) + j0) * C::kWideEb;
    const unsigned char *narrow = static_cast<const unsigned char *>(narrow_) + bh * N * int64_t(Dh) * (WIDE_CODED ? 2 : 1);
    const int fl = lane & 31, half = lane >> 5, blk = lane >> 4, sl = lane & 15;
    const int nchunks = (N + C::kCR - 1) / C::kCR;         // ANY: the last one may be ragged
    const int cols = N - j0 < C::kJW ? N - j0 : C::kJW;    // columns of this tile that exist (a multiple of 16, or any number)

    // ---- staging: a thread's vectors sit at the same place of every chunk ---------------------------------------------
    u32x4 wv[C::kAhead][C::kWideVecs], nv[C::kAhead][C::kNarrowVecs];
    int w_src[C::kWideVecs], w_dst[C::kWideVecs];          // byte offsets from the chunk's first row: in memory, in LDS
    constexpr int kV = 16 / C::kWideEb;
#pragma unroll
    for (int k = 0; k < C::kWideVecs; ++k) {
        const int v = tid + k * C::kNt, r = v / C::kVecRowW, cv = v % C::kVecRowW;
        // (a vector past the row's end: the row's first one; and one that the row ends in reads on into the next: columns past N
        // only reach sums that are never written)
        w_src[k] = (r * N + (cv * kV < cols ? cv * kV : -j0)) * C::kWideEb;
        w_dst[k] = r * C::kPitchW + cv * 16;
    }
    auto load_chunk = [&](int c, auto set_) {
        constexpr int S = decltype(set_)::value;
        const int left = N - c * C::kCR;                   // rows from the chunk's first one to the head's end
        const unsigned char *src = wide + int64_t(c) * C::kCR * N * C::kWideEb;
        const u32x4 *nsrc = reinterpret_cast<const u32x4 *>(narrow + int64_t(c) * C::kCR * Dh * (WIDE_CODED ? 2 : 1));
        if (left > C::kCR || (left == C::kCR && !last_head)) {   // uniform: the tensor goes on behind the chunk
#pragma unroll
            for (int k = 0; k < C::kWideVecs; ++k) {
                if constexpr (ANY) __builtin_memcpy(&wv[S][k], src + w_src[k], 16);
                else wv[S][k] = *reinterpret_cast<const u32x4 *>(src + w_src[k]);
            }
#pragma unroll
            for (int k = 0; k < C::kNarrowVecs; ++k) {
                const int v = tid + k * C::kNt;
                nv[S][k] = nsrc[v < C::kCR * C::kVecRowN ? v : 0];
            }
            return;
        }
        // rows past the end, and chunks past the end (RS > 1): zeros
#pragma unroll
        for (int k = 0; k < C::kWideVecs; ++k) {
            const int v = tid + k * C::kNt, r = v / C::kVecRowW, cv = v % C::kVecRowW;
            // (the vector that the tensor ends in: the tensor's last 16 bytes, moved to where they belong)
            const int over = ANY && r == left - 1 && cv * kV < cols && cv * kV + kV > cols ? (cv * kV + kV - cols) * C::kWideEb : 0;
            wv[S][k] = u32x4{0u, 0u, 0u, 0u};
            if (r < left) {
                if constexpr (ANY) {
                    __builtin_memcpy(&wv[S][k], src + w_src[k] - over, 16);
                    wv[S][k] = move_down(wv[S][k], over);
                } else {
                    wv[S][k] = *reinterpret_cast<const u32x4 *>(src + w_src[k]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < C::kNarrowVecs; ++k) {
            const int v = tid + k * C::kNt;
            nv[S][k] = v < (left < C::kCR ? left : C::kCR) * C::kVecRowN ? nsrc[v] : u32x4{0u, 0u, 0u, 0u};
        }
    };
    auto store_chunk = [&](int b, auto set_) {
        constexpr int S = decltype(set_)::value;
        unsigned char *lw = lds_tc + b * C::kStage, *ln = lw + C::kCR * C::kPitchW;
#pragma unroll
        for (int k = 0; k < C::kWideVecs; ++k) *reinterpret_cast<u32x4 *>(lw + w_dst[k]) = wv[S][k];
#pragma unroll
        for (int k = 0; k < C::kNarrowVecs; ++k) {
            const int v = tid + k * C::kNt;
            if (v < C::kCR * C::kVecRowN) *reinterpret_cast<u32x4 *>(ln + (v / C::kVecRowN) * C::kRowN + (v % C::kVecRowN) * 16) = nv[S][k];
        }
    };

    bm_v16f acc[C::kJB][DT];
    float dsum[DT];                                        // dV: column sums of dO for d = 32 dt + l%32 over this lane's rows
    float csum[C::kJB];                                    // dK: column sums of dS per j, per lane
#pragma unroll
    for (int jb = 0; jb < C::kJB; ++jb) {
        csum[jb] = 0.0f;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[jb][dt][v] = 0.0f;
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) dsum[dt] = 0.0f;
    // transposing reads: lane gets column (first column) + l%32 and the rows (first row) + 8*(l/32) ..+7
    const int wide_at = WIDE_CODED ? ((blk >> 1) * 8 + (sl >> 1)) * C::kPitchW + wave * 64 + (blk & 1) * 16 + (sl & 1) * 8
                                   : ((blk >> 1) * 8 + (sl >> 2)) * C::kPitchW + (wave * 64 + (blk & 1) * 16 + (sl & 3) * 4) * 2;
    const int narrow_at = WIDE_CODED ? ((blk >> 1) * 8 + (sl >> 2)) * C::kRowN + ((blk & 1) * 16 + (sl & 3) * 4) * 2
                                     : ((blk >> 1) * 8 + (sl >> 1)) * C::kRowN + (blk & 1) * 16 + (sl & 1) * 8;
    const bool wave_live = wave * 64 < cols;               // uniform per wave

    // the group's chunk c is the head's chunk c * RS + group; it waits in register set c % kAhead and goes to LDS buffer
    // c % 2 when chunk c - 1 is being multiplied
    const int steps = (nchunks + RS - 1) / RS;             // the same for every group: they meet at the barriers
    auto chunk_step = [&](int c, auto set_) {
        const int b = c & 1;
        store_chunk(b, set_);
        if (c + C::kAhead < steps) load_chunk((c + C::kAhead) * RS + group, set_);
        __syncthreads();   // chunk c is in LDS; every wave has finished with chunk c - 1 (the other buffer)
        const unsigned char *lw = lds_tc + b * C::kStage, *ln = lw + C::kCR * C::kPitchW;
        if (!wave_live) return;                          // its columns lie past N (the barrier above is still met)
#pragma unroll
        for (int ks = 0; ks < C::kCR / 16; ++ks) {
            bm_v8h fn[DT];
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                if (WIDE_CODED) {
                    const unsigned char *p = ln + narrow_at + ks * 16 * C::kRowN + dt * 64;
                    const bm_v4h lo = __builtin_bit_cast(bm_v4h, __builtin_amdgcn_ds_read_tr16_b64_v4i16(BM_LDS3(bm_v4s, p)));
                    const bm_v4h hi = __builtin_bit_cast(bm_v4h, __builtin_amdgcn_ds_read_tr16_b64_v4i16(BM_LDS3(bm_v4s, p + 4 * C::kRowN)));
                    fn[dt] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                    for (int q = 0; q < 8; q += 2) dsum[dt] = BmNum<ET>::dot_ones(fn[dt][q], fn[dt][q + 1], dsum[dt]);
                } else {
                    fn[dt] = BmNum<ET>::codes8(__builtin_amdgcn_ds_read_tr8_b64_v2i32(BM_LDS3(bm_v2i, ln + narrow_at + ks * 16 * C::kRowN + dt * 32)));
                }
            }
#pragma unroll
            for (int jb = 0; jb < C::kJB; ++jb) {
                if (wave * 64 + jb * 32 >= cols) break;       // uniform per wave: blocks past N
                bm_v8h fw;
                if (WIDE_CODED) {
                    fw = BmNum<ET>::codes8(__builtin_amdgcn_ds_read_tr8_b64_v2i32(BM_LDS3(bm_v2i, lw + wide_at + ks * 16 * C::kPitchW + jb * 32)));
                } else {
                    const unsigned char *p = lw + wide_at + ks * 16 * C::kPitchW + jb * 64;
                    const bm_v4h lo = __builtin_bit_cast(bm_v4h, __builtin_amdgcn_ds_read_tr16_b64_v4i16(BM_LDS3(bm_v4s, p)));
                    const bm_v4h hi = __builtin_bit_cast(bm_v4h, __builtin_amdgcn_ds_read_tr16_b64_v4i16(BM_LDS3(bm_v4s, p + 4 * C::kPitchW)));
                    fw = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                    for (int k = 0; k < 8; k += 2) csum[jb] = BmNum<ET>::dot_ones(fw[k], fw[k + 1], csum[jb]);
                }
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) acc[jb][dt] = BmNum<ET>::mfma(fn[dt], fw, acc[jb][dt]);
            }
        }
    };
    load_chunk(group, std::integral_constant<int, 0>());
    if (C::kAhead == 2 && steps > 1) load_chunk(RS + group, std::integral_constant<int, C::kAhead - 1>());
    for (int c = 0; c < steps; c += C::kAhead) {
        chunk_step(c, std::integral_constant<int, 0>());
        if (C::kAhead == 2 && c + 1 < steps) chunk_step(c + 1, std::integral_constant<int, C::kAhead - 1>());
    }
    if constexpr (RS > 1) {
        // the groups' sums, one group after the other: a value per lane at a stride of the group's threads
        float *sums = reinterpret_cast<float *>(lds_all) + tid;
        auto each = [&](auto f) {
            int n = 0;
#pragma unroll
            for (int jb = 0; jb < C::kJB; ++jb)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) { float t = acc[jb][dt][v]; f(t, n++); acc[jb][dt][v] = t; }
#pragma unroll
            for (int jb = 0; jb < C::kJB; ++jb) f(csum[jb], n++);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) f(dsum[dt], n++);
        };
#pragma unroll 1
        for (int g = 1; g < RS; ++g) {
            __syncthreads();   // every wave is done with the chunks, or with the sums before
            if (group == g) each([&](float &x, int n) { sums[n * C::kNt] = x; });
            __syncthreads();
            if (group == 0) each([&](float &x, int n) { x += sums[n * C::kNt]; });
        }
    }

    // ---- epilogue: lane l, register v of a tile: d = 32*dt + 8*(v/4) + 4*(l/32) + v%4, row j = (tile's first) + l%32 ----
    const int h = int(bh % heads);
    const float s = alpha[h] / 255.0f;
    const float off = fmaf(BmNum<ET>::kCentre, s, beta[h]);
    float *dsums = reinterpret_cast<float *>(lds_all);     // dV: the sums of dO per d, for every lane to pick its four
    if (WIDE_CODED) {
        __syncthreads();                                   // every wave is done with the chunks
        if (group == 0 && wave == 0) {                     // (a live wave: column 0 of the tile always exists)
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                const float t = dsum[dt] + __shfl_xor(dsum[dt], 32);   // both halves of the rows
                if (half == 0) dsums[dt * 32 + fl] = t;
            }
        }
        __syncthreads();
    }
    if (group != 0) return;
#pragma unroll
    for (int jb = 0; jb < C::kJB; ++jb) {
        const int j = j0 + wave * 64 + jb * 32 + fl;
        float cs = 0.0f;
        if (!WIDE_CODED) cs = off * (csum[jb] + __shfl_xor(csum[jb], 32));
        if (j >= N) continue;
        _Float16 *po = out + (bh * N + j) * int64_t(Dh) + half * 4;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                bm_v4h o;
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const float add = WIDE_CODED ? off * dsums[dt * 32 + g * 8 + half * 4 + k] : cs;
                    o[k] = BmNum<ET>::round(scale * fmaf(s, acc[jb][dt][4 * g + k], add));
                }
                *reinterpret_cast<bm_v4h *>(po + dt * 32 + g * 8) = o;
            }
    }
}

// ---- dQ = scale * dS K_hat for long rows: one workgroup per head -------------------------------------------
// The head's K codes go to LDS once (rows j, zeros beyond N; fragments by transposing reads).  dS comes in
// chunks of 64 rows -- contiguous, merely element-aligned pieces that lie in LDS as they lie in memory -- the
// next chunk's vectors waiting in registers while a chunk is multiplied.  Wave w takes rows 32*(w&1) ..+31 of
// the chunk and the d tiles of half w>>1.  A lane's dS fragment (eight consecutive j of its row) starts at an
// arbitrary element of LDS: five aligned 4-byte reads, shifted into place (a misaligned 16-byte LDS read
// stalls the LDS for dozens of cycles).  The MFMA runs with the codes on the M side, so a lane ends up with one
// row i and runs of four consecutive d, and the beta term's row sum is a per-lane scalar.
// Dh == 32 * DT, DT even or 1 (each half takes DT/2 tiles; DT == 1: only the waves of half 0 multiply).
template <int DT> struct NnCfg {
    static constexpr int Dh = 32 * DT;
    static constexpr int kRowK = Dh + 32;                  // bytes per staged code row
    static constexpr int kTiles = DT >= 2 ? DT / 2 : 1;    // d tiles of 32 per wave
    static constexpr int kNt = DT >= 2 ? 256 : 128;        // threads: four waves, or two when there is one d tile
    static constexpr int kMaxVecs = 1792 / kNt;            // dS vectors per thread and chunk
    static size_t ds_bytes(int64_t N) { return (size_t(64) * N * 2 + 16 + 64 + 15) & ~size_t(15); }
    static size_t lds_bytes(int64_t N) { return ds_bytes(N) + size_t(ceil_div(N, 16)) * 16 * kRowK; }
};

template <int DT, typename ET>
__global__ __launch_bounds__(NnCfg<DT>::kNt, 3) void k_attn_nn(const _Float16 *__restrict__ dS, const int8_t *__restrict__ kq,
                                                         _Float16 *__restrict__ dQ, int N, int heads, float scale,
                                                         const float *__restrict__ alpha_k, const float *__restrict__ beta_k,
                                                         int ds_bytes, int64_t ds_elems)
{
    typedef NnCfg<DT> C;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_nn[];
    constexpr int Dh = C::Dh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t bh = blockIdx.x;
    unsigned char *lk = lds_nn + ds_bytes;
    const int fl = lane & 31, half = lane >> 5;
    const int nchunks = (N + 63) >> 6;

    u32x4 wv[C::kMaxVecs];
    int mis = 0, nvec = 0, whole = 0;
    int64_t ebase = 0;
    auto load_chunk = [&](int c) {
        const int i0 = c * 64;
        const int rows = N - i0 < 64 ? N - i0 : 64;
        const int64_t e0 = (bh * N + i0) * int64_t(N);
        mis = int(e0 & 7);
        ebase = e0 - mis;
        nvec = (mis + rows * N + 7) >> 3;
        whole = ds_elems - ebase >= int64_t(nvec) * 8 ? nvec : nvec - 1;   // the tensor's last vector may reach past its end
        const u32x4 *src = reinterpret_cast<const u32x4 *>(dS + ebase);
#pragma unroll
        for (int k = 0; k < C::kMaxVecs; ++k) {
            const int v = tid + k * C::kNt;
            if (v < whole) wv[k] = src[v];
        }
    };
    auto store_chunk = [&]() {
#pragma unroll
        for (int k = 0; k < C::kMaxVecs; ++k) {
            const int v = tid + k * C::kNt;
            if (v < whole) *reinterpret_cast<u32x4 *>(lds_nn + v * 16) = wv[k];
        }
        if (whole < nvec && tid < 8) {
            const int64_t g = ebase + int64_t(whole) * 8 + tid;
            reinterpret_cast<_Float16 *>(lds_nn)[whole * 8 + tid] = g < ds_elems ? dS[g] : (_Float16)0.0f;
        }
    };

    load_chunk(0);
    {   // the head's K codes: rows j of Dh bytes, rows N .. (a multiple of 16) zero
        const u32x4 *kvec = reinterpret_cast<const u32x4 *>(kq + bh * N * int64_t(Dh));
        constexpr int kVecRow = Dh / 16;
        const int kvecs = N * kVecRow, all = ((N + 15) & ~15) * kVecRow;
        for (int v = tid; v < all; v += C::kNt) {
            u32x4 w = {0u, 0u, 0u, 0u};
            if (v < kvecs) w = kvec[v];
            *reinterpret_cast<u32x4 *>(lk + (v / kVecRow) * C::kRowK + (v % kVecRow) * 16) = w;
        }
    }

    const int blk = lane >> 4, sl = lane & 15;
    const int i_loc = (wave & 1) * 32 + fl;                // row of the chunk
    const int d0 = (wave >> 1) * (DT >= 2 ? Dh / 2 : 0);
    const unsigned char *pk = lk + ((blk >> 1) * 8 + (sl >> 1)) * C::kRowK + d0 + (blk & 1) * 16 + (sl & 1) * 8;
    const unsigned *lds32 = reinterpret_cast<const unsigned *>(lds_nn);
    const int h = int(bh % heads);
    const float s = alpha_k[h] / 255.0f;
    const float off = fmaf(BmNum<ET>::kCentre, s, beta_k[h]);

    for (int c = 0; c < nchunks; ++c) {
        __syncthreads();                                   // the previous chunk has been multiplied
        const int mis_c = mis;
        store_chunk();
        if (c + 1 < nchunks) load_chunk(c + 1);
        __syncthreads();
        const int rows = N - c * 64 < 64 ? N - c * 64 : 64;
        if ((wave & 1) * 32 >= rows) continue;             // uniform per wave; the barriers are at the loop's top
        const int e_row = mis_c + (i_loc < rows ? i_loc : rows - 1) * N + half * 8;   // rows past the end repeat the last one
        const int shift = (e_row & 1) * 16;
        bm_v16f acc[C::kTiles];
#pragma unroll
        for (int t = 0; t < C::kTiles; ++t)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;
        float rsum = 0.0f;
        for (int j0 = 0; j0 < N; j0 += 16) {
            const int w0 = (e_row + j0) >> 1;
            unsigned w[5];
#pragma unroll
            for (int q = 0; q < 5; ++q) w[q] = lds32[w0 + q];
            bm_v4u f;
#pragma unroll
            for (int q = 0; q < 4; ++q) f[q] = __builtin_amdgcn_alignbit(w[q + 1], w[q], shift);
            if (j0 + 16 > N) {                             // uniform: the row's ragged end, zeros beyond it
                const int j = j0 + half * 8;
#pragma unroll
                for (int q = 0; q < 4; ++q) f[q] &= (j + 2 * q < N ? 0xffffu : 0u) | (j + 2 * q + 1 < N ? 0xffff0000u : 0u);
            }
            const bm_v8h fs = __builtin_bit_cast(bm_v8h, f);
#pragma unroll
            for (int q = 0; q < 8; q += 2)
                rsum = BmNum<ET>::dot_ones(fs[q], fs[q + 1], rsum);
#pragma unroll
            for (int t = 0; t < C::kTiles; ++t) {
                const bm_v8h fc = BmNum<ET>::codes8(__builtin_amdgcn_ds_read_tr8_b64_v2i32(BM_LDS3(bm_v2i, pk + j0 * C::kRowK + t * 32)));
                acc[t] = BmNum<ET>::mfma(fc, fs, acc[t]);
            }
        }
        rsum += __shfl_xor(rsum, 32);                      // both halves of the row's slots
        if (i_loc < rows) {
            // lane l, register v of a tile: d = 32*t + 8*(v/4) + 4*(l/32) + v%4, row i = l%32
            const float add = off * rsum;
            _Float16 *po = dQ + (bh * N + c * 64 + i_loc) * int64_t(Dh) + d0 + half * 4;
#pragma unroll
            for (int t = 0; t < C::kTiles; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    bm_v4h o;
#pragma unroll
                    for (int k = 0; k < 4; ++k) o[k] = BmNum<ET>::round(scale * fmaf(s, acc[t][4 * g + k], add));
                    *reinterpret_cast<bm_v4h *>(po + t * 32 + g * 8) = o;
                }
        }
    }
}

// ---- dQ by tiles of rows: a workgroup takes 64 rows i of one head and walks along the columns ----
// j in chunks of 64 (larger chunks cost workgroups per CU, which cost more than the shorter row segments): per chunk 64
// row segments of dS (16-byte vectors, from any element) and the chunk's rows of K codes, both in LDS row by row, the next two
// chunks' vectors waiting in registers (two LDS buffers, one barrier per chunk).  Wave w takes rows 32 (w & 1) ..+31 and the d tiles of parity w >> 1.  A lane's dS fragment (its row, eight
// consecutive j) is one aligned 16-byte LDS read; the codes come through the byte-transposing read.  Codes on the M
// side as in k_attn_nn: a lane ends up with one row i and runs of four consecutive d.  dS is read exactly once.
template <int DT> struct NrCfg {
    static constexpr int Dh = 32 * DT;
    static constexpr int kJC = 64;                         // columns per chunk
    static constexpr int kPitchS = kJC * 2 + 16;           // bytes per staged row segment of dS: 16 (mod 128), eight rows' reads on different banks
    static constexpr int kRowK = Dh + 32;                  // bytes per staged code row
    static constexpr int kTiles = (DT + 1) / 2;
    static constexpr int kVecRowS = kJC / 8, kVecRowK = Dh / 16;
    static constexpr int kSVecs = 64 * kVecRowS / kThreads, kKVecs = (kJC * kVecRowK + kThreads - 1) / kThreads;
    static constexpr int kStage = 64 * kPitchS + kJC * kRowK;
    static constexpr int kLds = 2 * kStage;
    static constexpr int kAhead = 2;                       // chunks in registers ahead of the one in LDS
};

template <int DT, bool ANY, typename ET>
__global__ __launch_bounds__(kThreads, 2) void k_attn_nn_rows(const _Float16 *__restrict__ dS, const int8_t *__restrict__ kq,
                                                              _Float16 *__restrict__ dQ, int N, int heads, int tiles_i, int turns,
                                                              float scale, const float *__restrict__ alpha_k, const float *__restrict__ beta_k)
{
    typedef NrCfg<DT> C;
    __shared__ __attribute__((aligned(16))) unsigned char lds_nr[C::kLds];
    constexpr int Dh = C::Dh;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned bid = xcd_block(blockIdx.x, gridDim.x);
    const int64_t bh = bid / unsigned(tiles_i);
    const int i0 = int(bid % unsigned(tiles_i)) * 64;
    const int rows = N - i0 < 64 ? N - i0 : 64;
    const int fl = lane & 31, half = lane >> 5, blk = lane >> 4, sl = lane & 15;
    const int nchunks = (N + C::kJC - 1) / C::kJC;
    const unsigned char *srow = reinterpret_cast<const unsigned char *>(dS + (bh * N + i0) * int64_t(N));
    const unsigned char *krow = reinterpret_cast<const unsigned char *>(kq + bh * N * int64_t(Dh));

    u32x4 sv[C::kAhead][C::kSVecs], kv[C::kAhead][C::kKVecs];
    int s_src[C::kSVecs];                                  // byte offsets from the chunk's first column; rows past the end repeat the last one
#pragma unroll
    for (int k = 0; k < C::kSVecs; ++k) {
        const int v = tid + k * kThreads, r = v / C::kVecRowS;
        s_src[k] = ((r < rows ? r : rows - 1) * N + (v % C::kVecRowS) * 8) * 2;
    }
    // turns (nn_rows_turns): the row tiles of a head start at sixteen places and come round.  By the tile and not the workgroup: a head's sums are taken in the same order wherever
    // it stands in the batch.
    const int start = turns ? i0 / 64 % 16 * nchunks / 16 : 0;
    auto load_chunk = [&](int c, auto set_) {
        constexpr int S = decltype(set_)::value;
        c += start;
        if (c >= nchunks) c -= nchunks;
        const int j0 = c * C::kJC;
        const int cols = N - j0 < C::kJC ? N - j0 : C::kJC;   // a multiple of 8, or (ANY) any number
        const unsigned char *src = srow + int64_t(j0) * 2;
        if (cols == C::kJC) {                              // uniform
#pragma unroll
            for (int k = 0; k < C::kSVecs; ++k) {
                if constexpr (ANY) __builtin_memcpy(&sv[S][k], src + s_src[k], 16);
                else sv[S][k] = *reinterpret_cast<const u32x4 *>(src + s_src[k]);
            }
        } else {
            // columns past N: zeros
#pragma unroll
            for (int k = 0; k < C::kSVecs; ++k) {
                const int cv = (tid + k * kThreads) % C::kVecRowS, some = cols - cv * 8;
                sv[S][k] = u32x4{0u, 0u, 0u, 0u};
                if (some >= 8) {
                    if constexpr (ANY) __builtin_memcpy(&sv[S][k], src + s_src[k], 16);
                    else sv[S][k] = *reinterpret_cast<const u32x4 *>(src + s_src[k]);
                } else if (ANY && some > 0) {              // the row's last 16 bytes, moved to where they belong
                    __builtin_memcpy(&sv[S][k], src + s_src[k] - (8 - some) * 2, 16);
                    sv[S][k] = move_down(sv[S][k], (8 - some) * 2);
                }
            }
        }
        const u32x4 *ksrc = reinterpret_cast<const u32x4 *>(krow + int64_t(j0) * Dh);
#pragma unroll
        for (int k = 0; k < C::kKVecs; ++k) {
            const int v = tid + k * kThreads;
            kv[S][k] = v < cols * C::kVecRowK ? ksrc[v] : u32x4{0u, 0u, 0u, 0u};
        }
    };
    auto store_chunk = [&](int b, auto set_) {
        constexpr int S = decltype(set_)::value;
        unsigned char *ls = lds_nr + b * C::kStage, *lk = ls + 64 * C::kPitchS;
#pragma unroll
        for (int k = 0; k < C::kSVecs; ++k) {
            const int v = tid + k * kThreads;
            *reinterpret_cast<u32x4 *>(ls + (v / C::kVecRowS) * C::kPitchS + (v % C::kVecRowS) * 16) = sv[S][k];
        }
#pragma unroll
        for (int k = 0; k < C::kKVecs; ++k) {
            const int v = tid + k * kThreads;
            if (v < C::kJC * C::kVecRowK) *reinterpret_cast<u32x4 *>(lk + (v / C::kVecRowK) * C::kRowK + (v % C::kVecRowK) * 16) = kv[S][k];
        }
    };

    const int i_loc = (wave & 1) * 32 + fl;
    const int tpar = wave >> 1;                            // this wave's d tiles: tpar, tpar + 2, ..  (DT == 1: only parity 0 multiplies)
    const bool wave_live = (wave & 1) * 32 < rows && (DT >= 2 || tpar == 0);
    const int s_at = i_loc * C::kPitchS + half * 16;
    const int k_at = ((blk >> 1) * 8 + (sl >> 1)) * C::kRowK + (blk & 1) * 16 + (sl & 1) * 8 + tpar * 32;
    bm_v16f acc[C::kTiles];
#pragma unroll
    for (int t = 0; t < C::kTiles; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.0f;
    float rsum = 0.0f;

    // chunk c waits in register set c % 2; it goes to LDS buffer c % 2 when chunk c - 1 is being multiplied
    auto chunk_step = [&](int c, auto set_) {
        const int b = c & 1;
        store_chunk(b, set_);
        if (c + C::kAhead < nchunks) load_chunk(c + C::kAhead, set_);
        __syncthreads();   // chunk c is in LDS; every wave has finished with chunk c - 1 (the other buffer)
        if (!wave_live) return;
        const unsigned char *ls = lds_nr + b * C::kStage, *lk = ls + 64 * C::kPitchS;
        const int cols = start || N - c * C::kJC > C::kJC ? C::kJC : N - c * C::kJC;
#pragma unroll
        for (int ks = 0; ks < C::kJC / 16; ++ks) {
            if (ks * 16 >= cols) break;                    // uniform; a last step of eight columns multiplies zeros in its second half
            const bm_v8h fs = *reinterpret_cast<const bm_v8h *>(ls + s_at + ks * 32);
#pragma unroll
            for (int q = 0; q < 8; q += 2) rsum = BmNum<ET>::dot_ones(fs[q], fs[q + 1], rsum);
#pragma unroll
            for (int t = 0; t < C::kTiles; ++t) {
                if (DT % 2 == 1 && DT > 1 && tpar + 2 * t >= DT) break;   // uniform per wave
                const bm_v8h fc = BmNum<ET>::codes8(__builtin_amdgcn_ds_read_tr8_b64_v2i32(BM_LDS3(bm_v2i, lk + k_at + ks * 16 * C::kRowK + t * 64)));
                acc[t] = BmNum<ET>::mfma(fc, fs, acc[t]);
            }
        }
    };
    load_chunk(0, std::integral_constant<int, 0>());
    if (nchunks > 1) load_chunk(1, std::integral_constant<int, 1>());
    for (int c = 0; c < nchunks; c += 2) {
        chunk_step(c, std::integral_constant<int, 0>());
        if (c + 1 < nchunks) chunk_step(c + 1, std::integral_constant<int, 1>());
    }
    if (!wave_live) return;
    rsum += __shfl_xor(rsum, 32);                          // both halves of the row's slots
    if (i_loc < rows) {
        // lane l, register v of a tile: d = 32*(tile) + 8*(v/4) + 4*(l/32) + v%4, row i = l%32
        const int h = int(bh % heads);
        const float s = alpha_k[h] / 255.0f;
        const float add = fmaf(BmNum<ET>::kCentre, s, beta_k[h]) * rsum;
        _Float16 *po = dQ + (bh * N + i0 + i_loc) * int64_t(Dh) + tpar * 32 + half * 4;
#pragma unroll
        for (int t = 0; t < C::kTiles; ++t)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                if (DT % 2 == 1 && DT > 1 && tpar + 2 * t >= DT) break;
                bm_v4h o;
#pragma unroll
                for (int k = 0; k < 4; ++k) o[k] = BmNum<ET>::round(scale * fmaf(s, acc[t][4 * g + k], add));
                *reinterpret_cast<bm_v4h *>(po + t * 64 + g * 8) = o;
            }
    }
}

static bool nn_rows_fits(int64_t batches, int64_t N, int64_t Dh)
{
    if (Dh != 32 && Dh != 64 && Dh != 96 && Dh != 128) return false;
    return N >= 64 && batches * ceil_div(N, 64) < (int64_t(1) << 31);
}

// Whether the row tiles of a head start at different columns.  Rows of a multiple of 2 KB put the same columns of all rows on the same memory channels, where workgroups in
// step met: dQ and dK on new inputs each time (16, 1, 4096, 64) 215 -> 196 us, (36, 1, 2048, 64) 143 -> 130, (64, 1, 2048, 32) 211 -> 195, the whole attention backward 561 -> 543,
// 368 -> 356, 557 -> 542, of (7, 1, 6144, 64) 726 -> 718, (16, 1, 3072, 64) 332 -> 331.  A larger dS gains by the memory-side cache what workgroups in step leave there for each other: 670 MB
// (20, 1, 4096, 64) 265 -> 258, 805 MB (96, 1, 2048, 64) 318 -> 310 and (24, 1, 4096, 64) 314 -> 316, above (32, 1, 4096, 64) 385 -> 392, (128, 1, 2048, 64) 406 -> 413, (128, 1, 4096, 64) 1564 -> 1587.
// Rows of other multiples of 64, and of 1024, gain nothing: 1088 to 2112 -1 to +1 %, shorter ones up to 2 % behind.
static bool nn_rows_turns(int64_t batches, int64_t N) { return N % 1024 == 0 && N >= 2048 && batches * N * N * 2 <= 750000000; }

template <typename ET>
static void launch_nn_rows(const _Float16 *dS, const int8_t *kq, _Float16 *dQ, int64_t batches, int N, int Dh, int heads, float scale,
                           const float *alpha_k, const float *beta_k, hipStream_t s)
{
    const int tiles_i = int(ceil_div(N, 64)), turns = nn_rows_turns(batches, N);
    const dim3 grid(unsigned(batches * tiles_i));
#define MESA_LAUNCH_NR(DT_, ANY_) \
    hipLaunchKernelGGL((k_attn_nn_rows<DT_, ANY_, ET>), grid, dim3(kThreads), 0, s, dS, kq, dQ, N, heads, tiles_i, turns, scale, alpha_k, beta_k)
#define MESA_LAUNCH_NR_A(DT_) do { if (N % 8 == 0) MESA_LAUNCH_NR(DT_, false); else MESA_LAUNCH_NR(DT_, true); } while (0)
    if (Dh == 32) MESA_LAUNCH_NR_A(1);
    else if (Dh == 64) MESA_LAUNCH_NR_A(2);
    else if (Dh == 96) MESA_LAUNCH_NR_A(3);
    else MESA_LAUNCH_NR_A(4);
#undef MESA_LAUNCH_NR_A
#undef MESA_LAUNCH_NR
}

// whether k_attn_da can take the shape, and in which mode
static bool da_solo(int64_t batches, int64_t N) { return N <= 64 && batches * ceil_div(N, 32) < (int64_t(1) << 32); }
template <int KS> static bool da_fits(int64_t batches, int64_t N) { return DaCfg<KS>::lds_bytes(N, da_solo(batches, N)) <= 65536; }

template <int KS, typename ET> static void launch_da(const _Float16 *dO, const int8_t *vq, _Float16 *dA, int64_t batches, int N, int heads,
                                        const float *alpha_v, const float *beta_v, hipStream_t s)
{
    typedef DaCfg<KS> C;
    const int codes_at = int(C::codes_at(N));
    if (da_solo(batches, N)) {
        const int64_t items = batches * ceil_div(N, 32);
        hipLaunchKernelGGL((k_attn_da<KS, true, ET>), dim3(unsigned(ceil_div(items, C::kWaves))), dim3(kThreads), C::lds_bytes(N, true), s, dO,
                           vq, dA, N, heads, alpha_v, beta_v, int64_t(0), codes_at, unsigned(items));
        return;
    }
    const unsigned gx = unsigned(ceil_div(N, 32));
    for (int64_t b0 = 0; b0 < batches; b0 += 65535) {   // the y extent of a grid is limited to 65535
        const int64_t nb = batches - b0 < 65535 ? batches - b0 : 65535;
        hipLaunchKernelGGL((k_attn_da<KS, false, ET>), dim3(gx, unsigned(nb)), dim3(kThreads), C::lds_bytes(N, false), s, dO, vq, dA, N,
                           heads, alpha_v, beta_v, b0, codes_at, 0u);
    }
}

// whether k_attn_tn can take the shape; a chunk of 32 rows is then within kMaxWideVecs vectors per thread, and all of it within the 64 KiB of LDS
// that a kernel gets by default
static bool tn_fits(int64_t N, int64_t Dh) { return (Dh == 32 || Dh == 64 || Dh == 96 || Dh == 128) && N < 128; }

template <int DT, bool WIDE_CODED, int NW, typename ET>
static void launch_tn_one(const void *wide, const void *narrow, _Float16 *out, int64_t batches, int N, int heads, float scale,
                          const float *alpha, const float *beta, hipStream_t s)
{
    typedef TnCfg<DT, WIDE_CODED, NW> C;
    hipLaunchKernelGGL((k_attn_tn<DT, WIDE_CODED, NW, ET>), dim3(unsigned(batches)), dim3(C::kNt), C::lds_bytes(N), s, wide, narrow,
                       out, N, heads, scale, alpha, beta, int(C::wide_bytes(N)), batches * N * int64_t(N));
}

template <bool WIDE_CODED, typename ET>
static void launch_tn(const void *wide, const void *narrow, _Float16 *out, int64_t batches, int N, int Dh, int heads, float scale,
                      const float *alpha, const float *beta, hipStream_t s)
{
    // a wave per block of 32 rows j
#define MESA_TN(DT_) \
    do { \
        if (N <= 32) launch_tn_one<DT_, WIDE_CODED, 1, ET>(wide, narrow, out, batches, N, heads, scale, alpha, beta, s); \
        else if (N <= 64) launch_tn_one<DT_, WIDE_CODED, 2, ET>(wide, narrow, out, batches, N, heads, scale, alpha, beta, s); \
        else launch_tn_one<DT_, WIDE_CODED, 4, ET>(wide, narrow, out, batches, N, heads, scale, alpha, beta, s); \
    } while (0)
    if (Dh == 32) MESA_TN(1);
    else if (Dh == 64) MESA_TN(2);
    else if (Dh == 96) MESA_TN(3);
    else MESA_TN(4);
#undef MESA_TN
}

// whether k_attn_nn can take the shape: a 64-row chunk of dS within kMaxVecs vectors per thread, LDS within 64 KiB
// by tiles: k_attn_da_cols
static bool da_cols_fits(int64_t batches, int64_t N, int64_t Dh)
{
    if (Dh != 32 && Dh != 64 && Dh != 96 && Dh != 128) return false;
    // from 64 on: below, at most one of a workgroup's four waves has columns (N = 48: 0.28 against 0.24 ms for N = 49 through k_attn_da)
    return N >= 64 && batches * ceil_div(N, 256) * ceil_div(N, 64) < (int64_t(1) << 31);   // 64: the fewest rows a workgroup takes
}

// Whether a dA by tiles leaves non-temporally.  Kept like other lines it pushes the operands out of the L2s and leaves these, some at a time, during the kernels
// that follow; but one that the memory-side cache would take in wants to go there.  The whole attention backward on new inputs each time, each side behind itself (behind
// a call of the other, a kept result is written back at that one's cost), kept -> non-temporal us:
// Rows of a multiple of 128 elements, which meet on the same memory channels: (458, 256, 64) 97 -> 101, (114, 512, 64) 91 -> 96, (104, 640, 64) 129 -> 132, (29, 1024, 64) 98 -> 101,
// at 135 to 165 MB (286, 512, 64) 202 -> 204, (84, 896, 64) 184 -> 187, (72, 1024, 64) 202 -> 204, (79, 1024, 64) 213 -> 216, (183, 640, 64) 208 -> 204, (16, 2048, 64) 182 -> 183, above (1297, 256, 64) 254 -> 250,
// (576, 384, 64) 256 -> 251, (106, 896, 64) 219 -> 216, (105, 1024, 64) 272 -> 265, (26, 2048, 64) 263 -> 257, dV, dA and softmax of (16, 4096, 64) 407 -> 363; of 128 elements
// (1831, 128, 64), 60 MB, 131 -> 132, (2594, 128, 64) 176 and 176, (3072, 128, 64), 101 MB, 209 -> 206, (3662, 128, 64) 245 -> 243, (3662, 128, 32) 179 -> 180, (4578, 128, 64) 305 -> 299.
// Rows on half lines: (62, 448, 64) 53.0 -> 50.7, (101, 352, 64) 58.6 -> 57.0, (122, 320, 32) 48.4 -> 46.4, (541, 608, 64) 559 -> 533, (179, 1056, 64) 507 -> 480; shorter ones
// (399, 224, 64) 78.7 -> 81.3, (1562, 160, 64) 162 -> 166, (2170, 96, 64) 113 -> 117.  About half of the memory-side cache is better kept: 115 to 145 MB
// (120, 736, 64) 182 -> 187, (74, 992, 64) 202 -> 210, (65, 1056, 64) 206 -> 211, (282, 480, 32) 168 -> 174, (29, 1568, 64) 192 -> 196; at 100 and 160 MB (51, 992, 64) 148 -> 149, (81, 992, 64)
// 221 -> 217, of longer rows still (18, 2080, 64) 211 -> 218, (14, 2528, 64), 179 MB, 239 -> 242, at 190 MB (22, 2080, 64) 248 -> 241; but not at up to 448 elements ((324, 448, 64)
// 189 -> 182, (562, 320, 32) 155 -> 151) or wider heads ((131, 704, 96) 212 -> 206, (166, 576, 128) 219 and 219).
// Rows that start elsewhere end in parts of lines: (51, 1, 656, 64) 88 -> 95, (428, 1, 176, 32) 52 -> 56.
static bool da_streams(int64_t batches, int64_t N, int64_t Dh)
{
    const int64_t bytes = batches * N * N * 2;
    if (N % 128 == 0) return bytes >= (N == 128 ? 100000000 : 170000000);
    if (N % 32 != 0 || N < 256) return false;
    return Dh > 64 || N <= 448 || bytes <= 105000000 || bytes >= (N < 1536 ? 155000000 : 180000000);
}

template <typename ET>
static void launch_da_cols(const _Float16 *dO, const int8_t *vq, _Float16 *dA, int64_t batches, int N, int Dh, int heads,
                           const float *alpha_v, const float *beta_v, hipStream_t s)
{
    const int streams = da_streams(batches, N, Dh);
#define MESA_LAUNCH_DC(KS_) \
    do { \
        const int tiles_j = int(ceil_div(N, 256)), tiles_i = int(ceil_div(N, DcCfg<KS_>::kRows)); \
        const dim3 grid(unsigned(batches * tiles_j * tiles_i)); \
        if (N % 8 == 0) hipLaunchKernelGGL((k_attn_da_cols<KS_, false, ET>), grid, dim3(kThreads), 0, s, dO, vq, dA, N, heads, tiles_j, tiles_i, streams, alpha_v, beta_v); \
        else hipLaunchKernelGGL((k_attn_da_cols<KS_, true, ET>), grid, dim3(kThreads), 0, s, dO, vq, dA, N, heads, tiles_j, tiles_i, streams, alpha_v, beta_v); \
    } while (0)
    if (Dh == 32) MESA_LAUNCH_DC(2);
    else if (Dh == 64) MESA_LAUNCH_DC(4);
    else if (Dh == 96) MESA_LAUNCH_DC(6);
    else MESA_LAUNCH_DC(8);
#undef MESA_LAUNCH_DC
}

// by tiles: k_attn_tn_cols
static bool tn_cols_fits(int64_t batches, int64_t N, int64_t Dh)
{
    if (Dh != 32 && Dh != 64 && Dh != 96 && Dh != 128) return false;
    return N >= 64 && batches * ceil_div(N, 256) < (int64_t(1) << 31);
}

template <bool WIDE_CODED, typename ET>
static void launch_tn_cols(const void *wide, const void *narrow, _Float16 *out, int64_t batches, int N, int Dh, int heads, float scale,
                           const float *alpha, const float *beta, hipStream_t s)
{
    const int tiles_j = int(ceil_div(N, 256));
    const int64_t wgs = batches * tiles_j;
    // groups per workgroup, by the workgroups there are: (1, 16, 4096, 64), 256 of them, 759 / 644 / 630 us for the whole
    // attention backward with 1 / 2 / 4 groups; (2, 16, 4096, 64), 512: 1269 / 1235 / 1251; (8, 12, 1024, 64), 384:
    // 261 / 254 / 265; (16, 12, 576, 64), 576: 188 / 200 / 210.  At heads of 96 and 128 two groups fill a CU's registers, and more workgroups than CUs take a
    // second round: dA and dV with two groups -> one, (275, 256, 96) 35.3 -> 30.2 us, (313, 140, 96) 26.7 -> 20.8, (374, 64, 128) 18.8 -> 12.0.  Below 128 rows a
    // group has four chunks or fewer and the adding costs more than it saves: (366, 112, 64) 15.3 -> 14.2, dQ and dK 14.0 -> 13.0.
    const int rs = N < 128 || wgs > (Dh <= 64 ? 512 : 256) ? 1 : wgs <= 256 && N >= 1024 && Dh <= 64 ? 4 : 2;
#define MESA_LAUNCH_TC(DT_, RS_) \
    do { \
        const dim3 grid{unsigned(wgs)}, block(TcCfg<DT_, WIDE_CODED, RS_>::kNt * (RS_)); \
        if (N % 16 == 0) hipLaunchKernelGGL((k_attn_tn_cols<DT_, WIDE_CODED, RS_, false, ET>), grid, block, 0, s, wide, narrow, out, N, heads, tiles_j, scale, alpha, beta); \
        else hipLaunchKernelGGL((k_attn_tn_cols<DT_, WIDE_CODED, RS_, true, ET>), grid, block, 0, s, wide, narrow, out, N, heads, tiles_j, scale, alpha, beta); \
    } while (0)
    if (Dh == 32) { if (rs == 4) MESA_LAUNCH_TC(1, 4); else if (rs == 2) MESA_LAUNCH_TC(1, 2); else MESA_LAUNCH_TC(1, 1); }
    else if (Dh == 64) { if (rs == 4) MESA_LAUNCH_TC(2, 4); else if (rs == 2) MESA_LAUNCH_TC(2, 2); else MESA_LAUNCH_TC(2, 1); }
    else if (Dh == 96) { if (rs == 2) MESA_LAUNCH_TC(3, 2); else MESA_LAUNCH_TC(3, 1); }
    else { if (rs == 2) MESA_LAUNCH_TC(4, 2); else MESA_LAUNCH_TC(4, 1); }
#undef MESA_LAUNCH_TC
}

static bool nn_fits(int64_t N, int64_t Dh)
{
    if (Dh != 32 && Dh != 64 && Dh != 128) return false;
    if ((64 * N + 14) / 8 + 1 > 1792) return false;
    const int64_t ds = (64 * N * 2 + 16 + 64 + 15) / 16 * 16;
    return ds + ceil_div(N, 16) * 16 * (Dh + 32) <= 65536;
}

template <int DT, typename ET> static void launch_nn(const _Float16 *dS, const int8_t *kq, _Float16 *dQ, int64_t batches, int N, int heads,
                                        float scale, const float *alpha_k, const float *beta_k, hipStream_t s)
{
    typedef NnCfg<DT> C;
    hipLaunchKernelGGL((k_attn_nn<DT, ET>), dim3(unsigned(batches)), dim3(C::kNt), C::lds_bytes(N), s, dS, kq, dQ, N, heads, scale,
                       alpha_k, beta_k, int(C::ds_bytes(N)), batches * N * int64_t(N));
}

// Which kernel a product of 16-bit tensors takes: the general one, the one that goes by tiles of columns or rows, or the one that keeps a
// head's rows or codes whole.  The lines lie where some thousands of shapes put them (1 to 2500 heads, 8 to 9000 tokens); us of the product
// alone, by the general kernel / by tiles / whole, where a path exists.  What decides is how many workgroups a way of cutting leaves: the
// general kernel has a workgroup per 64 x 64 results and its loads are its own, the others share what they read.
enum AttnWay { kWayGeneral, kWayTiles, kWayWhole };

// dA.  Whole: 32 x N results in LDS.  Aligned rows by tiles once these give the CUs enough workgroups -- the more of a tile's 256 columns exist, the fewer
// will do: general / by tiles / whole, calls of dA and dV, (118, 224, 64), 236 workgroups, 16.5 / 14.5 / 19.5, (12, 760, 64), 216, 18.4 / 17.0 / 18.8, (6, 728, 128), 216,
// 16.6 / 14.5 / 17.0, (9, 544, 64), 135, +1.0 by tiles, (64, 64, 64) +0.5 --, else whole, but not where N is a multiple of 32, whose rows meet on the same banks
// ((192, 256, 64): +15).  Wide heads of less than 96 rows whole: (403, 80, 96) 22.5 / 20.7 / 18.3, (822, 72, 96) 30.0 / 27.4 / 24.3.  Unaligned rows whole up to 800 tokens ((192, 301, 64)
// -6.6 by tiles, -9.1 whole; (192, 420, 64) -17.0 and -17.7; (27, 553, 64) 20.5 / 21.3 / 18.2, (42, 463, 128) 34.1 / 31.7 / 28.2, (44, 524, 64) - / 25.7 / 22.7, (18, 733, 64) - / 23.5 /
// 21.9), unless heads are few and long ((3, 420, 64) +0.9, (8, 511, 64) +0.4), or, beyond 448 tokens, many and the tiles well filled ((192, 577, 64) 4 us behind, (38, 687, 64) +1.1 of
// 31, (24, 765, 64) +1.6 of 27), or 96 wide (0 to +2: (37, 741, 96), (41, 655, 96)).
static AttnWay da_way(int64_t batches, int64_t N, int64_t Dh)
{
    const bool whole = (Dh == 32 && da_fits<2>(batches, N)) || (Dh == 64 && da_fits<4>(batches, N)) || (Dh == 96 && da_fits<6>(batches, N)) ||
                       (Dh == 128 && da_fits<8>(batches, N));
    const int64_t per_head = ceil_div(N, 256) * ceil_div(N, Dh <= 64 ? 128 : 64);
    const bool aligned = N % 8 == 0 && N >= 64;
    if (whole && aligned && N < 96 && N % 32 != 0 && Dh > 64) return kWayWhole;
    if (whole && !aligned) {
        if (N <= 256 || (N <= 448 && batches >= ceil_div(128, ceil_div(N, 32)))) return kWayWhole;
        const bool filled = 4 * N >= 3 * 256 * ceil_div(N, 256);   // the tiles' columns, three quarters of them
        const int64_t many = N > 704 ? 352 : Dh == 64 && filled ? 640 : 2048;
        if (N > 448 && N <= 800 && Dh != 96 && batches >= ceil_div(192, ceil_div(N, 32)) && batches < ceil_div(many, per_head)) return kWayWhole;
    }
    if (da_cols_fits(batches, N, Dh) && batches >= ceil_div(!aligned ? 384 : N > 448 ? 144 : N >= 192 ? 160 : 256, per_head)) return kWayTiles;
    return whole && aligned && N % 32 != 0 ? kWayWhole : kWayGeneral;
}

// dV and dK.  Both other ways give a workgroup all the rows of a head, so they want columns, some hundred per CU at Dh = 64, which the general
// kernel's tiles fit exactly, fewer at other sizes; a head of less than 32 rows costs what one of 32 does.  dV by tiles: (64, 301, 64) +1.3, (64, 577, 64) -3.2,
// (64, 919, 64) -18, (192, 197, 64) -1.9, (1536, 197, 96) -83; (3, 601, 64) +5.  Whole (a few percent ahead) below 128 tokens: (1536, 71, 64) dK -1.2 by tiles, -3.0
// whole; (1536, 131, 64) -11.6 and -11.1.  Whole against general, dK: (2048, 8, 128) 17.0 -> 11.8, (1536, 10, 128) -3.9, (1536, 12, 32) -2.1, (571, 33, 32) -0.7,
// (200, 23, 96) +0.1; dV of (275, 71, 32) -0.5, by tiles of (14, 1392, 32) -3.0, (29, 575, 32) -1.8, (132, 128, 96),
// 16896 columns, +1.7 of 11.1.  Heads of up to 32 rows are a wave each, of which some hundred do: calls of dQ and dK by the general kernel / whole, (582, 8, 128) 8.9 / 7.7, (450, 13, 96)
// 9.5 / 8.4, (733, 8, 64) 7.9 / 7.2, 256 heads of 64 or 96 -0.1 to -0.4, dA and dV -0.1 to +0.1 there, at heads of 128 +0.4 with 256 and 0.0 with 360.
static AttnWay tn_way(int64_t batches, int64_t N, int64_t Dh)
{
    const bool whole = tn_fits(N, Dh) && batches < (int64_t(1) << 31);
    const int64_t columns = N <= 32 && whole ? (Dh == 128 ? 11520 : 8192) : Dh == 32 ? 12288 : Dh == 64 ? 28672 : Dh == 96 ? 18432 : 20480;
    if (batches < ceil_div(columns, N < 32 ? 32 : N)) return kWayGeneral;
    if (tn_cols_fits(batches, N, Dh) && (N >= 128 || N % 16 == 0 || !whole)) return kWayTiles;
    return whole ? kWayWhole : kWayGeneral;
}

// dQ.  Whole, a workgroup per head, for many short heads whose rows do not meet on the same banks: (768, 197, 64) -3.8 by tiles, -4.4 whole;
// (3072, 100, 64) -1.3, -4.1 (with dK behind it, (768, 100, 64) 22.7 by the general kernel, 22.2); (1536, 100, 32) -1.6, -2.6; (1536, 150, 32) -4.1, -1.1; (768, 150, 128) -9, -14; (768, 197,
// 128) -24, -19; (8, 197, 64) 0 and +7; against tiles, (949, 125, 32) -1.9, (750, 118, 32) -1.7, (516, 97, 128) -3.0, aligned (1550, 80, 32) +5.9, (526, 144, 128) +5.7.  By tiles from 192 workgroups on ((192, 301, 96)
// -11, (24, 919, 96) -3.5, (8, 919, 96) +2.9), short heads only where the general kernel's 64 x 64 tiles do not fit Dh; always at Dh = 32, half such a tile ((64, 601, 32) -3.7, (192, 74, 32)
// -0.7).  Long heads fill the general kernel's workgroups well, so by tiles later: (16, 888, 96), 224 workgroups, +3.0, (11, 1126, 128), 198, +3.9, (14, 1426, 64), 322, +2.2, (19, 1356,
// 64), 418, +2.3; (55, 512, 64), 440, -1.0, (15, 1168, 128), 285, -2.1.
static AttnWay nn_way(int64_t batches, int64_t N, int64_t Dh)
{
    if (nn_fits(N, Dh) && batches < (int64_t(1) << 31)) {
        const bool many = Dh == 32 ? N % 8 != 0 && N < 144 && batches >= 640 : Dh == 64 ? batches >= 640 : N < 192 && batches >= (N % 8 != 0 ? 512 : 640);
        if (N < 64 || (N % 32 != 0 && many)) return kWayWhole;
    }
    if (!nn_rows_fits(batches, N, Dh)) return kWayGeneral;
    const int64_t enough = ceil_div(Dh == 64 ? (N < 704 ? 192 : 448) : N <= 448 ? 192 : 256, ceil_div(N, 64));
    const bool tiles = Dh == 32 || (batches >= enough && (Dh == 64 ? N >= 192 : Dh == 96 || N >= 128 || batches >= 384));
    return tiles ? kWayTiles : kWayGeneral;
}

static mesa_status check_attn(int64_t B, int64_t H, int64_t N, int64_t Dh, mesa_dtype dt)
{
    if (!valid_dtype(dt) || B < 0 || H < 0 || N < 0 || Dh < 0) return MESA_ERR_INVALID_ARG;
    if (N >= (int64_t(1) << 20) || Dh >= (int64_t(1) << 20)) return MESA_ERR_UNSUPPORTED;
    // 32-bit element offsets inside one (sample, head); the row / column tile counts fit a grid dimension
    if ((long double)N * (long double)N >= 2147483648.0L || (long double)N * (long double)Dh >= 2147483648.0L)
        return MESA_ERR_UNSUPPORTED;
    if ((long double)B * (long double)H >= 9.0e15L) return MESA_ERR_UNSUPPORTED;
    return MESA_OK;
}

}  // namespace mesa

using namespace mesa;

extern "C" MESA_EXPORT mesa_status mesa_attn_av_bwd_q(const int8_t *aq, const int8_t *vq, int64_t B, int64_t H, int64_t N,
                                                      int64_t Dh, const float *alpha_a, const float *beta_a,
                                                      const float *alpha_v, const float *beta_v, const void *dO, void *dA,
                                                      void *dV, mesa_dtype dt, void *stream)
{
    mesa_status st = check_attn(B, H, N, Dh, dt);
    if (st != MESA_OK) return st;
    if (B == 0 || H == 0 || N == 0 || Dh == 0) return MESA_OK;
    if (!aq || !vq || !dO || !dA || !dV || !alpha_a || !beta_a || !alpha_v || !beta_v) return MESA_ERR_INVALID_ARG;
    if (!aligned16(aq) || !aligned16(vq) || !aligned16(dO) || !aligned16(dA) || !aligned16(dV) || !aligned4(alpha_a) ||
        !aligned4(beta_a) || !aligned4(alpha_v) || !aligned4(beta_v))
        return MESA_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t batches = B * H;
    BmmArgs a{};
    a.heads = int(H);
    a.scale = 1.0f;
    // dA[i,j] = sum_d dO[i,d] * V_hat[j,d]:  P = dO (r = i, t = d),  Q = V (t = d, c = j)
    a.x = static_cast<const _Float16 *>(dO); a.y = vq; a.c = static_cast<_Float16 *>(dA);
    a.x_batch = N * Dh; a.y_batch = N * Dh; a.c_batch = N * N;
    a.R = int(N); a.Cn = int(N); a.Tn = int(Dh);
    a.p_rs = Dh; a.p_ts = 1; a.q_ts = 1; a.q_cs = Dh;
    a.alpha = alpha_v; a.beta = beta_v;
    // dV[j,d] = sum_i A_hat[i,j] * dO[i,d]:  P = A (r = j, t = i),  Q = dO (t = i, c = d)
    BmmArgs v = a;
    v.y = aq; v.c = static_cast<_Float16 *>(dV);
    v.y_batch = N * N; v.c_batch = N * Dh;
    v.R = int(N); v.Cn = int(Dh); v.Tn = int(N);
    v.p_rs = 1; v.p_ts = N; v.q_ts = Dh; v.q_cs = 1;
    v.alpha = alpha_a; v.beta = beta_a;
    if (N < 8 || Dh < 8) {   // an extent shorter than one load vector: the plain kernel
        launch_bmm_plain<false>(a, batches, dt, s);
        launch_bmm_plain<true>(v, batches, dt, s);
        return launch_status();
    }
    if (launch_bmm_waves_two<BmProduct<false, true, true>, BmProduct<true, false, false>>(a, v, batches, dt, s)) return launch_status();
#define MESA_AV_DA(ET) \
    do { \
        if (launch_bmm_waves<false, true, true, ET>(a, batches, s)) break; \
        const AttnWay way = da_way(batches, N, Dh); \
        if (way == kWayTiles) launch_da_cols<ET>(a.x, vq, a.c, batches, int(N), int(Dh), int(H), alpha_v, beta_v, s); \
        else if (way == kWayGeneral) launch_bmm<false, true, true, ET>(a, batches, s); \
        else if (Dh == 32) launch_da<2, ET>(a.x, vq, a.c, batches, int(N), int(H), alpha_v, beta_v, s); \
        else if (Dh == 64) launch_da<4, ET>(a.x, vq, a.c, batches, int(N), int(H), alpha_v, beta_v, s); \
        else if (Dh == 96) launch_da<6, ET>(a.x, vq, a.c, batches, int(N), int(H), alpha_v, beta_v, s); \
        else launch_da<8, ET>(a.x, vq, a.c, batches, int(N), int(H), alpha_v, beta_v, s); \
    } while (0)
    auto da = [&]() {
        if (dt == MESA_F32) {
            if (!launch_bmm_waves<false, true, true, float>(a, batches, s)) launch_bmm<false, true, true, float>(a, batches, s);
        } else if (dt == MESA_BF16) MESA_AV_DA(__bf16); else MESA_AV_DA(_Float16);
    };
#undef MESA_AV_DA
#define MESA_AV_DV(ET) \
    do { \
        if (launch_bmm_waves<true, false, false, ET>(v, batches, s)) break; \
        const AttnWay way = tn_way(batches, N, Dh); \
        if (way == kWayTiles) launch_tn_cols<true, ET>(aq, dO, v.c, batches, int(N), int(Dh), int(H), 1.0f, alpha_a, beta_a, s); \
        else if (way == kWayWhole) launch_tn<true, ET>(aq, dO, v.c, batches, int(N), int(Dh), int(H), 1.0f, alpha_a, beta_a, s); \
        else launch_bmm<true, false, false, ET>(v, batches, s); \
    } while (0)
    auto dv = [&]() {
        if (dt == MESA_F32) {
            if (!launch_bmm_waves<true, false, false, float>(v, batches, s)) launch_bmm<true, false, false, float>(v, batches, s);
        } else if (dt == MESA_BF16) MESA_AV_DV(__bf16); else MESA_AV_DV(_Float16);
    };
#undef MESA_AV_DV
    // dV, bound by its reads, goes first where dA is about as large as the memory-side cache (256 MB) and more: a dA just written is still leaving that cache
    // while the next kernel reads, and softmax behind it, which would find a smaller one there, finds little of this one.  The whole attention backward on new inputs each time,
    // dA first -> dV first us, kept: (315, 577, 64) 317 -> 306, (102, 1127, 64) 354 -> 337, (1680, 250, 64) 346 -> 341, (2706, 197, 64) 386 -> 385.  One that leaves non-temporally
    // (da_streams) gains as long as dO and the rest stay in reach, up to some 600000 rows: (8, 4096, 64) 331 -> 319, (16, 4096, 64) 580 -> 560, (66, 4096, 64) 2708 -> 2700,
    // (124, 1024, 64) 307 -> 297, (477, 1024, 64) 1212 -> 1202, (760, 544, 64) 658 -> 634, (1567, 288, 32) 385 -> 373; with more (1049, 1024, 64) 2692 -> 2715, (1221, 640, 64) 1288 -> 1299,
    // (2219, 352, 64) 860 -> 880, (3315, 288, 64) 944 -> 960; rows of up to 256 elements never: (1831, 256, 96) 410 -> 417, (6104, 256, 64) 1135 -> 1149, (14648, 128, 64) 905 -> 910.
    // binary32 either way at any size: (4, 12, 1024, 64), 201 MB, 285 -> 292, (1, 6, 4096, 64), 403 MB, 588 -> 582.
    const bool dv_first = dt != MESA_F32 && batches * N * N >= 115000000 && (!da_streams(batches, N, Dh) || (N > 256 && batches * N <= 600000));
    if (dv_first) {
        dv();
        da();
    } else {
        da();
        dv();
    }
    return launch_status();
}

extern "C" MESA_EXPORT mesa_status mesa_attn_qk_bwd_q(const int8_t *qq, const int8_t *kq, int64_t B, int64_t H, int64_t N,
                                                      int64_t Dh, const float *alpha_q, const float *beta_q,
                                                      const float *alpha_k, const float *beta_k, const void *dS, float scale,
                                                      void *dQ, void *dK, mesa_dtype dt, void *stream)
{
    mesa_status st = check_attn(B, H, N, Dh, dt);
    if (st != MESA_OK) return st;
    if (!(scale == scale)) return MESA_ERR_INVALID_ARG;
    if (B == 0 || H == 0 || N == 0 || Dh == 0) return MESA_OK;
    if (!qq || !kq || !dS || !dQ || !dK || !alpha_q || !beta_q || !alpha_k || !beta_k) return MESA_ERR_INVALID_ARG;
    if (!aligned16(qq) || !aligned16(kq) || !aligned16(dS) || !aligned16(dQ) || !aligned16(dK) || !aligned4(alpha_q) ||
        !aligned4(beta_q) || !aligned4(alpha_k) || !aligned4(beta_k))
        return MESA_ERR_INVALID_ARG;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t batches = B * H;
    BmmArgs a{};
    a.heads = int(H);
    a.scale = scale;
    a.x = static_cast<const _Float16 *>(dS);
    a.x_batch = N * N; a.y_batch = N * Dh; a.c_batch = N * Dh;
    a.R = int(N); a.Cn = int(Dh); a.Tn = int(N);
    // dQ[i,d] = scale * sum_j dS[i,j] * K_hat[j,d]:  P = dS (r = i, t = j),  Q = K (t = j, c = d)
    a.y = kq; a.c = static_cast<_Float16 *>(dQ);
    a.p_rs = N; a.p_ts = 1; a.q_ts = Dh; a.q_cs = 1;
    a.alpha = alpha_k; a.beta = beta_k;
    // dK[j,d] = scale * sum_i dS[i,j] * Q_hat[i,d]:  P = dS (r = j, t = i),  Q = Q codes (t = i, c = d)
    BmmArgs k = a;
    k.y = qq; k.c = static_cast<_Float16 *>(dK);
    k.p_rs = 1; k.p_ts = N; k.q_ts = Dh; k.q_cs = 1;
    k.alpha = alpha_q; k.beta = beta_q;
    if (N < 8 || Dh < 8) {
        launch_bmm_plain<false>(a, batches, dt, s);
        launch_bmm_plain<false>(k, batches, dt, s);
        return launch_status();
    }
    if (launch_bmm_waves_two<BmProduct<false, true, false>, BmProduct<false, false, false>>(a, k, batches, dt, s)) return launch_status();
#define MESA_QK_DQ(ET) \
    do { \
        const AttnWay way = nn_way(batches, N, Dh); \
        if (way == kWayTiles) launch_nn_rows<ET>(a.x, kq, a.c, batches, int(N), int(Dh), int(H), scale, alpha_k, beta_k, s); \
        else if (way == kWayGeneral) launch_bmm<false, true, false, ET>(a, batches, s); \
        else if (Dh == 32) launch_nn<1, ET>(a.x, kq, a.c, batches, int(N), int(H), scale, alpha_k, beta_k, s); \
        else if (Dh == 64) launch_nn<2, ET>(a.x, kq, a.c, batches, int(N), int(H), scale, alpha_k, beta_k, s); \
        else launch_nn<4, ET>(a.x, kq, a.c, batches, int(N), int(H), scale, alpha_k, beta_k, s); \
    } while (0)
    if (dt == MESA_F32) launch_bmm<false, true, false, float>(a, batches, s);
    else if (dt == MESA_BF16) MESA_QK_DQ(__bf16); else MESA_QK_DQ(_Float16);
#undef MESA_QK_DQ
#define MESA_QK_DK(ET) \
    do { \
        const AttnWay way = tn_way(batches, N, Dh); \
        if (way == kWayTiles) launch_tn_cols<false, ET>(dS, qq, k.c, batches, int(N), int(Dh), int(H), scale, alpha_q, beta_q, s); \
        else if (way == kWayWhole) launch_tn<false, ET>(dS, qq, k.c, batches, int(N), int(Dh), int(H), scale, alpha_q, beta_q, s); \
        else launch_bmm<false, false, false, ET>(k, batches, s); \
    } while (0)
    if (dt == MESA_F32) launch_bmm<false, false, false, float>(k, batches, s);
    else if (dt == MESA_BF16) MESA_QK_DK(__bf16); else MESA_QK_DK(_Float16);
#undef MESA_QK_DK
    return launch_status();
}

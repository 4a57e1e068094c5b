// softmax_rows.hpp -- what the two row-per-lane-group softmax kernels (forward with quantizer, backward at
// de-quantized codes) share: the tile shape, the wave-level synchronisation, reductions inside a lane group and
// the staged element's conversions.
//
// Rows of an attention map (197, 49 elements) start at odd byte offsets.  A wave owns a tile of R consecutive rows
// with R * cols a multiple of 8, i.e. a run of whole 8-element vectors that is 16-byte aligned in the tensors and
// 8-byte aligned in the codes: memory is only touched as whole aligned vectors (flat phases), the tile lies in the
// wave's LDS region as it lies in memory, and in between a row belongs to a group of LPR lanes, lane l holding
// elements l, l + LPR, ... in EPL register slots, each a constant distance from the lane's first element.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"
#include "quantize.hpp"

namespace mesa {

template <int TPT> __device__ __forceinline__ void team_sync()
{
    if (TPT == kThreads) {
        __syncthreads();
    } else {   // the team is one wave: order its own LDS traffic
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

constexpr int kSrTileElems = 2048;                    // elements of a wave's tile at most
constexpr int kSrFlat = kSrTileElems / kVec / 64;     // vectors per lane in the flat phases
constexpr int kSrMaxCols = 256;
constexpr int kSrSlack = 1024;                        // bytes past the last region that unused slots may read

template <int WIDTH, bool MAX> __device__ __forceinline__ float lanes_extreme_dpp(float v)
{
    static_assert(WIDTH == 8 || WIDTH == 16 || WIDTH == 32 || WIDTH == 64, "aligned power-of-two lane groups");
    v = MAX ? vmax(v, dpp_move<0xB1>(v)) : vmin(v, dpp_move<0xB1>(v));      // quad_perm [1,0,3,2]
    v = MAX ? vmax(v, dpp_move<0x4E>(v)) : vmin(v, dpp_move<0x4E>(v));      // quad_perm [2,3,0,1]
    v = MAX ? vmax(v, dpp_move<0x141>(v)) : vmin(v, dpp_move<0x141>(v));    // row_half_mirror
    if (WIDTH >= 16) v = MAX ? vmax(v, dpp_move<0x140>(v)) : vmin(v, dpp_move<0x140>(v));   // row_mirror
    if (WIDTH >= 32) { const float o = __shfl_xor(v, 16, 64); v = MAX ? vmax(v, o) : vmin(v, o); }
    if (WIDTH >= 64) { const float o = __shfl_xor(v, 32, 64); v = MAX ? vmax(v, o) : vmin(v, o); }
    return v;
}

// one staged element <-> binary32; put() returns the value as stored
template <typename T> struct LdsElem;

// v rounded to the storage type
template <typename T> __device__ __forceinline__ float as_stored(float v) { return float(T(v)); }
template <> __device__ __forceinline__ float as_stored<float>(float v) { return v; }
template <> struct LdsElem<_Float16> {
    __device__ static __forceinline__ float get(const unsigned char *p) { return float(*reinterpret_cast<const _Float16 *>(p)); }
    __device__ static __forceinline__ float put(unsigned char *p, float v)
    {
        const _Float16 h = _Float16(v);
        *reinterpret_cast<_Float16 *>(p) = h;
        return float(h);
    }
};
template <> struct LdsElem<__bf16> {
    __device__ static __forceinline__ float get(const unsigned char *p)
    {
        return __uint_as_float(uint32_t(*reinterpret_cast<const uint16_t *>(p)) << 16);
    }
    __device__ static __forceinline__ float put(unsigned char *p, float v)
    {
        const __bf16 h = __bf16(v);
        const uint16_t bits = __builtin_bit_cast(uint16_t, h);
        *reinterpret_cast<uint16_t *>(p) = bits;
        return __uint_as_float(uint32_t(bits) << 16);
    }
};
template <> struct LdsElem<float> {
    __device__ static __forceinline__ float get(const unsigned char *p) { return *reinterpret_cast<const float *>(p); }
    __device__ static __forceinline__ float put(unsigned char *p, float v)
    {
        *reinterpret_cast<float *>(p) = v;
        return v;
    }
};

// lanes per row, slots per lane and rows per tile for rows of `cols` <= kSrMaxCols elements
struct SrShape {
    int lpr, epl;
    bool tight;          // cols > lpr * (epl - 1): only a lane's last slot can lie beyond the row's end
    int64_t R, tiles;
};

inline SrShape sr_shape(int64_t total_rows, int64_t cols)
{
    SrShape p{};
    if (cols <= 56) { p.lpr = 8; p.epl = 7; }
    else if (cols <= 64) { p.lpr = 8; p.epl = 8; }         // 8 x 8 windows: every slot used (8 x 13 leaves 38 % idle)
    else if (cols <= 104) { p.lpr = 8; p.epl = 13; }
    else if (cols <= 128) { p.lpr = 8; p.epl = 16; }
    else if (cols <= 200) { p.lpr = 8; p.epl = 25; }
    else { p.lpr = 16; p.epl = 16; }
    p.tight = cols > int64_t(p.lpr) * (p.epl - 1);
    int64_t gc = cols, b8 = 8;
    while (b8) { int64_t t = gc % b8; gc = b8; b8 = t; }
    const int64_t unit = 8 / gc, rpp = 64 / p.lpr;
    const int64_t step = unit > rpp ? unit : rpp;          // whole vectors per tile, whole passes
    p.R = (kSrTileElems / cols) / step * step;             // step * cols <= 8 * 256
    if (p.R > total_rows) p.R = (total_rows + step - 1) / step * step;
    p.tiles = (total_rows + p.R - 1) / p.R;
    return p;
}

// ---------------------------------------------------------------------------------------------
// Long rows that start anywhere (256 < cols <= 2048, cols no multiple of 8).  The same three phases, but a tile is as
// large as its alignment asks for -- eight rows of an odd length, 4616 elements at 577 columns -- and belongs to a
// workgroup (two or four waves in the forward, four or eight in the backward), whose waves share out its vectors, then its
// rows, then its vectors; a row takes half a wave or a whole one.  The forward's workgroups stride over the tiles and request the
// next one's first vectors while they work; the backward has a workgroup per tile, and the CU's other workgroups cover
// the latency.  (A tile per wave was measured first: half the waves per CU fit their LDS, and a small tensor's few tiles take
// four times as long each -- 30 against 19 us at three maps of 587 columns.)
// ---------------------------------------------------------------------------------------------
constexpr int64_t kSlMaxCols = 2048;
constexpr int64_t kSlTileElems = 6144;                 // several units of rows per tile up to here

// slots that every row of a shape fills (the shape before it ends there)
constexpr int sl_full(int epl) { return epl == 12 ? 8 : epl == 16 ? 12 : epl == 20 ? 16 : epl == 24 ? 20 : 24; }

struct SlPlan {
    bool ok;
    int lpr, epl;
    int64_t R, tiles;
    int waves;               // per workgroup
    uint32_t tab_bytes;
    size_t lds;
};

// tab: bytes of the workgroup's tables; elem: bytes of a tile per element
inline SlPlan sl_plan(int64_t total_rows, int64_t cols, int64_t tab, int64_t elem, int waves)
{
    SlPlan p{};
    if (cols <= kSrMaxCols || cols > kSlMaxCols || cols % kVec == 0) return p;
    p.lpr = cols <= 1024 ? 32 : 64;
    const int64_t slots = (cols + p.lpr - 1) / p.lpr;
    p.epl = slots <= 12 ? 12 : slots <= 16 ? 16 : slots <= 20 ? 20 : slots <= 24 ? 24 : 32;
    const int64_t unit = cols % 4 == 0 ? 2 : cols % 2 == 0 ? 4 : 8;   // rows until a row starts on a vector boundary again
    const int64_t units = kSlTileElems / (unit * cols);
    p.R = unit * (units > 1 ? units : 1);
    if (p.R > total_rows) p.R = (total_rows + unit - 1) / unit * unit;
    p.tiles = (total_rows + p.R - 1) / p.R;
    p.tab_bytes = uint32_t((tab + 15) / 16 * 16);
    // behind the tile: what the last row's unused slots may read
    p.lds = size_t(p.tab_bytes) + size_t((p.R * cols * elem + 15) / 16 * 16) + size_t(p.lpr) * p.epl * 4;
    if (p.lds > 64 * 1024) return p;
    p.waves = waves;
    p.ok = true;
    return p;
}

// expands X(LPR, EPL) with the shape of plan p
#define MESA_FOR_SL_SHAPE(p, X) \
    do { \
        if ((p).lpr == 32) { \
            if ((p).epl == 12) X(32, 12); \
            else if ((p).epl == 16) X(32, 16); \
            else if ((p).epl == 20) X(32, 20); \
            else if ((p).epl == 24) X(32, 24); \
            else X(32, 32); \
        } else { \
            if ((p).epl == 20) X(64, 20); \
            else if ((p).epl == 24) X(64, 24); \
            else X(64, 32); \
        } \
    } while (0)

}  // namespace mesa

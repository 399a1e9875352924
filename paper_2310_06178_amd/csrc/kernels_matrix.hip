// The matrix form of msgemm_run: Y = M x X with the codes decoded in registers and the sums done by the matrix cores.
//
// The two phases of the method add, for every row, the table entries L(codes, j) = sum_r b(i_r) x(jd + r) that its
// codes address (Section 3.2, second line of the y(i) equation).  Where the matrix cores are the adders, the entries
// need not be tabulated first: sum_j sum_r b(i_r) x(jd + r) is the first line of the same equation, and one
// v_mfma_f32_16x16x32 forms and adds the entries of 16 rows x 16 groups of two codes x 16 columns at once.  Nothing is
// built per workgroup, so a workgroup can own its rows for all of k: there are no partial sums between workgroups, no
// second launch and no table start-up, and the kernel is bound by the code stream.  Values, products and sums are those
// of the full-width tables: the integers -8..7 are exact in fp16 / bf16 / int8, products are exact, sums are fp32
// (int32 for int8 activations).
//
// The plan's rule (matrix_choose_shape) gives this form what the library chooses itself for the paper's encoding at
// d = 2, and 8-bit weights whose value map is a format the device converts (E4M3, E5M2, times a power of two); tables in
// LDS remain for every request for a variant, other value maps and scale blocks that are not whole runs of 128 columns.
//
// Layout of the codes: [row group of 16 R rows][run of 128 columns][row tile r < R][lane][16 bytes].  Lane (n, q) =
// (lane & 15, lane >> 4) holds columns 32 q + 0..31 of row n of its tile, dword w of its 16 bytes the 8 from 8 w on, with
// the nibbles in the order the decoder yields them; MFMA step t takes dword t of every lane (int8: dwords 2 t, 2 t + 1).
// One 16-byte load of a wavefront is 1 KiB of consecutive memory and one row tile's share of a run.
// Scales: [row group][scale block][n][r] fp16, so a lane's scales for its R tiles are one load.
// The tile kernel's tiles have 32 rows: lane (n, h) = (lane & 31, lane >> 5) holds columns 64 h + 0..63 of row n in two such loads, one behind the
// other (8-bit codes: four); its steps take 8 columns of each half (int8: 16).
#include "device_types.h"
#include "fused_common.h"
#include "msgemm_internal.h"

#include <math.h>

#include <algorithm>
#include <iterator>
#include <type_traits>

namespace msgemm {
namespace {

constexpr int kRun = 128;          // columns of k per step: one 16-byte load per lane and row tile
constexpr uint32_t kPastEnd = 0x7fff0000u;  // a buffer offset past any plan's codes: the load returns zero and reads nothing
constexpr int kTileRowWaves = 2;   // tile kernel: wavefronts side by side in rows
constexpr int kAuxNt = 2;          // buffer cache policy bit: non-temporal (every code is used once)

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef int v16i __attribute__((ext_vector_type(16)));

// 16 bytes at any alignment the element type allows (columns of X may start anywhere)
template <int kAlign> struct __attribute__((packed, aligned(kAlign))) Any16 { uint32_t a, b, c, d; };

template <int kAlign> __device__ __forceinline__ v4u load_any16(const void* p)
{
    const Any16<kAlign> v = *(const Any16<kAlign>*)p;
    return v4u{v.a, v.b, v.c, v.d};
}
template <int kAlign> struct __attribute__((packed, aligned(kAlign))) Any4 { uint32_t a; };
struct __attribute__((packed, aligned(1))) Any2 { uint16_t a; };

// What differs between the activation types.
//   kFrags  operand registers (16 bytes) of X per run of 128 columns and tile of 16 columns of X; one MFMA each
//   kRaw    16-byte loads per run as X is stored
//   decode  the codes of one MFMA step -> its weight operand
template <typename XT> struct Policy;

// (x & mask) | bits in one instruction: with `bits` as a constant the compiler takes two, so its value is hidden from it.  (The
// instruction itself is left to the compiler.  Written as inline asm it is not looked at when the wait states behind a matrix
// instruction are counted, and its result may take a register that the matrix instruction has yet to write.)
__device__ __forceinline__ uint32_t and_or(uint32_t x, uint32_t mask, uint32_t bits)
{
    asm("" : "+v"(bits));
    return (x & mask) | bits;
}

template <> struct Policy<__half> {
    using acc_t = v4f;
    using out_t = __half;
    static constexpr int kFrags = 4, kRaw = 4;
    static __device__ __forceinline__ void decode(const v4u& c, int t, v4u& w)
    {
        // offset-binary nibbles: 0x6400 | u is 1024 + u in fp16 (and 1024 + 16 u with the nibble one place up); the
        // offset is taken off exactly (adding an integer's bits to those of a large power of two is an old and widely published
        // way to convert it)
        const uint32_t x = c[t], y = x >> 8;
        const v2h off0 = {(_Float16)-1032.0f, (_Float16)-1032.0f}, off1 = {(_Float16)-72.0f, (_Float16)-72.0f};
        const v2h sixteenth = {(_Float16)0.0625f, (_Float16)0.0625f};
        const v2h a = __builtin_bit_cast(v2h, and_or(x, 0x000f000fu, 0x64006400u)) + off0;
        const v2h b = __builtin_bit_cast(v2h, and_or(x, 0x00f000f0u, 0x64006400u)) * sixteenth + off1;
        const v2h d = __builtin_bit_cast(v2h, and_or(y, 0x000f000fu, 0x64006400u)) + off0;
        const v2h e = __builtin_bit_cast(v2h, and_or(y, 0x00f000f0u, 0x64006400u)) * sixteenth + off1;
        w = v4u{__builtin_bit_cast(uint32_t, a), __builtin_bit_cast(uint32_t, b), __builtin_bit_cast(uint32_t, d),
                __builtin_bit_cast(uint32_t, e)};
    }
    static __device__ __forceinline__ v4f mma(const v4u& x, const v4u& w, const v4f& c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, x), __builtin_bit_cast(v8h, w), c, 0, 0, 0);
    }
};

struct Bf16Weights {
    static __device__ __forceinline__ void decode(const v4u& c, int t, v4u& w)
    {
        // two's-complement nibbles: v_cvt_off_f32_i4 gives value / 16 in fp32, whose upper half is its bf16; the factor
        // is a power of two and is put back with the sums
        const uint32_t x = c[t];
        uint32_t y = x >> 4;
        // (hidden, or the compiler takes bits 12 to 19 of x instead of byte 1 of y, which the conversion cannot select by itself: an instruction more for
        // three of the eight)
        asm("" : "+v"(y));
        const float f0 = __builtin_amdgcn_cvt_off_f32_i4((int)x), f1 = __builtin_amdgcn_cvt_off_f32_i4((int)((x >> 8) & 0xff));
        const float f2 = __builtin_amdgcn_cvt_off_f32_i4((int)((x >> 16) & 0xff)), f3 = __builtin_amdgcn_cvt_off_f32_i4((int)(x >> 24));
        const float f4 = __builtin_amdgcn_cvt_off_f32_i4((int)y), f5 = __builtin_amdgcn_cvt_off_f32_i4((int)((y >> 8) & 0xff));
        const float f6 = __builtin_amdgcn_cvt_off_f32_i4((int)((y >> 16) & 0xff)), f7 = __builtin_amdgcn_cvt_off_f32_i4((int)(y >> 24));
        w = v4u{__builtin_amdgcn_perm(__float_as_uint(f1), __float_as_uint(f0), 0x07060302u),
                __builtin_amdgcn_perm(__float_as_uint(f3), __float_as_uint(f2), 0x07060302u),
                __builtin_amdgcn_perm(__float_as_uint(f5), __float_as_uint(f4), 0x07060302u),
                __builtin_amdgcn_perm(__float_as_uint(f7), __float_as_uint(f6), 0x07060302u)};
    }
    static __device__ __forceinline__ v4f mma(const v4u& x, const v4u& w, const v4f& c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, x), __builtin_bit_cast(v8bf, w), c, 0, 0, 0);
    }
};

template <> struct Policy<bf16_t> : Bf16Weights {
    using acc_t = v4f;
    using out_t = bf16_t;
    static constexpr int kFrags = 4, kRaw = 4;
};

// fp32 activations: x = h + m + l in three bf16 pieces of eight bits each (see Split), three MFMAs per step.
template <> struct Policy<float> : Bf16Weights {
    using acc_t = v4f;
    using out_t = float;
    static constexpr int kFrags = 4, kRaw = 8;
};

template <> struct Policy<int8_t> {
    using acc_t = v4i;
    using out_t = int;
    static constexpr int kFrags = 2, kRaw = 2;
    static __device__ __forceinline__ void decode(const v4u& c, int t, v4u& w)
    {
        // two's-complement nibbles in the upper half of a byte are 16 x the value; the sums are shifted back
        w = v4u{(c[2 * t] << 4) & 0xf0f0f0f0u, c[2 * t] & 0xf0f0f0f0u, (c[2 * t + 1] << 4) & 0xf0f0f0f0u,
                c[2 * t + 1] & 0xf0f0f0f0u};
    }
    static __device__ __forceinline__ v4i mma(const v4u& x, const v4u& w, const v4i& c)
    {
        return __builtin_amdgcn_mfma_i32_16x16x64_i8(__builtin_bit_cast(v4i, x), __builtin_bit_cast(v4i, w), c, 0, 0, 0);
    }
};

// 8-bit codes of a floating-point format the device converts (every finite pattern exact in fp16 and bf16): two dwords of
// four codes -> the weight operand of one MFMA step.
enum Format { kInt4, kE4M3, kE5M2 };
// times a power of two (bf16 only, whose range has room for it: the products are then those of the map's own values)
template <int F, typename XT, bool kHigh> __device__ __forceinline__ uint32_t convert_pair(uint32_t x, float times)
{
    if constexpr (__is_same(XT, __half)) {
        if constexpr (F == kE4M3) return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8((int)x, 1.0f, kHigh));
        else return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_bf8((int)x, 1.0f, kHigh));
    } else {
        if constexpr (F == kE4M3) return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8((int)x, times, kHigh));
        else return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_bf8((int)x, times, kHigh));
    }
}
template <int F, typename XT> __device__ __forceinline__ v4u convert(uint32_t lo, uint32_t hi, float times)
{
    return v4u{convert_pair<F, XT, false>(lo, times), convert_pair<F, XT, true>(lo, times),
               convert_pair<F, XT, false>(hi, times), convert_pair<F, XT, true>(hi, times)};
}

// Which nibble of a code dword holds the e-th of its 8 columns, and what is stored there for a two's-complement code.
enum Encoding { kEncF16, kEncBf16, kEncI8 };
__host__ __device__ __forceinline__ int nibble_of(int enc, int e)
{
    if (enc == kEncF16) return (e >> 1 & 1) | (e >> 2 & 1) << 1 | (e & 1) << 2;  // pairs (0,4) (1,5) (2,6) (3,7)
    return e < 4 ? 2 * e : 2 * (e - 4) + 1;                                     // low nibbles of the bytes, then high ones
}
__host__ __device__ __forceinline__ uint32_t stored_code(int enc, uint32_t code) { return enc == kEncF16 ? code ^ 8u : code; }
inline int encoding_of(int x_dtype)
{
    return x_dtype == MSGEMM_F16 ? kEncF16 : x_dtype == MSGEMM_I8 ? kEncI8 : kEncBf16;
}

struct MatrixArgs {
    const uint8_t* codes;
    const __half* scales;
    const void* X;
    int64_t ldx;
    void* Y;
    int64_t ldy;
    int64_t m, k;
    int b;                 // columns of X
    int runs;              // ceil(k / 128)
    int full_runs;         // k / 128
    int nblocks;           // scale blocks per row
    FastDiv div_block;     // runs per scale block
    uint32_t* partials;    // several k-segments: [segment][column][row of m_pad] fp32 / int32, else nullptr
    int64_t m_pad;
    int seg_runs;          // full runs per segment (tile kernel: runs)
    int row_groups;
    int passes;            // passes over the columns of X
    float factor;          // a power of two that the weight operands leave out (bf16 activations, 4-bit codes: value / 16;
                           // fp16 activations, 8-bit codes: the map's, which could take the weights out of fp16's range)
    float times;           // a power of two that the weight operands have in them (8-bit codes, bf16 and fp32 activations)
};

// fp32 activations: four elements as the three bf16 parts x = h + m + l, eight bits each by truncation.  Exact but for two
// kinds of elements, which the kernel makes up for after its loop (`split` takes six instructions an element in it):
//   * bf16 ends at 2^-133, so the last part of an element under 2^-109 may lose bits.  The lower half of `lost` tells whether
//     one did; split_lost gives those bits, 2^64 times as large, in the same form.
//   * An infinity leaves a NaN in the second part, and so in every sum of its column.  split_any takes the differences from
//     the element clamped to the finite range: an infinite activation is then infinite in its first part and adds finite
//     numbers in the others (as it does in a fp32 product), and a NaN is made quiet first (the upper half of one whose
//     payload lies in the lower sixteen bits only would be that of an infinity).
template <typename XT> constexpr int kOperands = sizeof(XT) == 4 ? 3 : 1;
struct Split { v2u part[3]; };
constexpr float kLostUp = 0x1p64f, kLostUnit = 0x1p-64f;
__device__ __forceinline__ uint32_t upper_halves(uint32_t lo, uint32_t hi) { return __builtin_amdgcn_perm(hi, lo, 0x07060302u); }
__device__ __forceinline__ float upper_half(uint32_t v) { return __uint_as_float(v & 0xffff0000u); }
__device__ __forceinline__ void split_finite(const v4u& x, const v4u& first, Split& s, uint32_t (&l)[4])
{
    uint32_t m[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        m[e] = __float_as_uint(__uint_as_float(x[e]) - upper_half(x[e]));
        l[e] = __float_as_uint(__uint_as_float(m[e]) - upper_half(m[e]));
    }
    s.part[0] = v2u{upper_halves(first[0], first[1]), upper_halves(first[2], first[3])};
    s.part[1] = v2u{upper_halves(m[0], m[1]), upper_halves(m[2], m[3])};
    s.part[2] = v2u{upper_halves(l[0], l[1]), upper_halves(l[2], l[3])};
}
__device__ __forceinline__ void split(const v4u& x, Split& s, uint32_t& lost)
{
    uint32_t l[4];
    split_finite(x, x, s, l);
    lost |= l[0] | l[1] | l[2] | l[3];
    asm volatile("" : "+v"(lost));   // (here and now: the compiler would keep all these until the end of the loop)
}
__device__ __forceinline__ void split_any(v4u x, Split& s, uint32_t (&l)[4])
{
    v4u v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        x[e] = __float_as_uint(__builtin_canonicalizef(__uint_as_float(x[e])));
        v[e] = __float_as_uint(__builtin_amdgcn_fmed3f(__uint_as_float(x[e]), -3.402823466e38f, 3.402823466e38f));
    }
    split_finite(v, x, s, l);
}
__device__ __forceinline__ void split_lost(const v4u& x, Split& s)
{
    uint32_t l[4], none[4];
    split_any(x, s, l);
    v4u y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = __float_as_uint((__uint_as_float(l[e]) - upper_half(l[e])) * kLostUp);
    split_finite(y, y, s, none);
}

// LDS only: the loads in flight to registers are not waited for
__device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Streaming kernel.  A workgroup owns 16 R rows for all of k; its W wavefronts take the runs of 128 columns in turn, each
// with D runs of codes and activations in flight, and add their sums through LDS.  Bound by the code stream.  Wavefronts
// share nothing until the end, so there is no barrier in the loop; activations come straight from the L2.
//
// kCols4 > 0, up to 4 kCols4 columns of X: consecutive lanes load consecutive 16-byte pieces of a column (a lane holding
// the operand of a column of its own instead would touch 64 cache lines per load, which the L1 takes one by one), and the
// wavefront passes them through an LDS buffer of its own into operand order: lane (n, q) then has column n.
// kCols4 == 0, up to four columns (int8: eight): lane n loads column n / T for step n % T of a run only (T steps) -- one
// load, nothing to transpose -- and every step has accumulators of its own, of which the rows of that step are the ones
// that count.  They end up in the same lane: y(column q) is the sum over t of register t of accumulator t of lane group q.
//
// Measured (one launch in a graph, cold codes; in brackets the table kernels with their second launch where they have
// one): 16384 x 4096 x 1 fp16 7.4 us = 4.5 TB/s (9.5; a launch that only reads the codes 6.7), 49152 x 12288 x 1 44.7 us =
// 6.8 TB/s (51.7), 14336 x 4096 x 16 fp16 with scales 8.9 us (30), 8192 x 8192 x 16 int8 8.0 us (30), 4096 x 4096 x 4 fp32
// 5.3 us (8.9), 8192 x 8192 E4M3 codes, one column, 12.9 us (18.0).  Without decoding and products the first takes 7.1, without
// its activations 7.5.  What is left at sixteen columns is the way of the activations through the LDS, as many bytes as of
// codes, and the decoding: two to three vector instructions per pair of weights against one MFMA for sixteen columns.
template <typename XT, int R, int kCols4, int W, int D, bool kScaled, int F>
__global__ void __launch_bounds__(W * 64)
matrix_stream_kernel(MatrixArgs a)
{
    using P = Policy<XT>;
    using acc_t = typename P::acc_t;
    using YT = typename P::out_t;
    constexpr bool kInt = sizeof(XT) == 1;
    constexpr bool kCompact = kCols4 == 0;
    constexpr int T = P::kFrags;
    constexpr int kOps = kOperands<XT>;
    constexpr int kPiece = 16 / (int)sizeof(XT);       // elements of a 16-byte piece
    constexpr int kLanesPerCol = kRun / kPiece;        // pieces of a column's run
    constexpr int kColsPerLoad = 64 / kLanesPerCol;
    constexpr int kRaw = kCompact ? P::kRaw / T : (4 * kCols4 + kColsPerLoad - 1) / kColsPerLoad;
    constexpr int kAcc = kCompact ? T : 1;             // accumulators per row tile
    constexpr int kRows = 16 * R;
    constexpr int kPitch = kRows + 4;                  // LDS: the four lane groups' columns fall on different banks
    constexpr int kCols = kCompact ? 16 / T : 4 * kCols4; // columns of X the kernel holds
    constexpr int kXWords = kCompact ? 0 : kOps * T * 256; // a wavefront's operands of one run
    constexpr int kRedWords = W * kCols * kPitch;
    __shared__ __align__(16) uint32_t lds[W * kXWords > kRedWords ? W * kXWords : kRedWords];

    int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, q = lane >> 4;
    const int rg = blockIdx.x;
    const int col0 = blockIdx.z * kCols;               // passes of kCols columns
    const int ncols = a.b - col0 < kCols ? a.b - col0 : kCols;

    constexpr int kVecs = F == kInt4 ? 1 : 2;          // 16-byte loads of codes per lane, row tile and run
    constexpr uint32_t run_bytes = R * kVecs * 1024u;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.codes + (int64_t)rg * a.runs * run_bytes), 0, (int)(a.runs * run_bytes), 0x00020000);
    const __amdgpu_buffer_rsrc_t srsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.scales + (int64_t)rg * a.nblocks * kRows), 0, kScaled ? (int)(a.nblocks * kRows * 2) : 0, 0x00020000);

    // where this lane's pieces of a run of X start (columns past the last one repeat it: their sums are not used), and
    // which column of the run the first element is
    int first;
    const XT* xcol[kCompact ? 1 : kRaw];
    auto locate = [&] {
        first = kCompact ? 32 * (lane >> 4) + (lane & 15) % T * (kInt ? 16 : 8) : lane % kLanesPerCol * kPiece;
#pragma unroll
        for (int i = 0; i < (kCompact ? 1 : kRaw); ++i) {
            int c = kCompact ? (lane & 15) / T : i * kColsPerLoad + lane / kLanesPerCol;
            c = c < ncols ? c : ncols - 1;
            xcol[i] = (const XT*)a.X + (int64_t)(col0 + c) * a.ldx + first;
        }
    };
    locate();

    struct Stage {
        v4u codes[R * kVecs];
        v4u x[kRaw];
        uint32_t q[(R + 1) / 2];
    };

    auto load_codes_of = [&](Stage& st, int run, bool ok) {
        const uint32_t off = (ok ? (uint32_t)run * run_bytes : kPastEnd) + lane * 16u;
#pragma unroll
        for (int r = 0; r < R * kVecs; ++r)
            st.codes[r] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(off + r * 1024u), 0, kAuxNt);
        if constexpr (kScaled) {
            const uint32_t so = fast_div((uint32_t)(ok ? run : 0), a.div_block) * (uint32_t)(kRows * 2) + n * (uint32_t)(R * 2);
            if constexpr (R == 4) {
                const v2u v = __builtin_amdgcn_raw_buffer_load_b64(srsrc, (int)so, 0, 0);
                st.q[0] = v.x; st.q[1] = v.y;
            } else if constexpr (R == 2) {
                st.q[0] = __builtin_amdgcn_raw_buffer_load_b32(srsrc, (int)so, 0, 0);
            } else {
                st.q[0] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(srsrc, (int)so, 0, 0);
            }
        }
    };
    auto piece_of = [&](int i) { return kCompact ? xcol[0] + i * kPiece : xcol[kCompact ? 0 : i]; };
    auto load_x = [&](Stage& st, int run) {
#pragma unroll
        for (int i = 0; i < kRaw; ++i) st.x[i] = load_any16<sizeof(XT)>(piece_of(i) + (int64_t)run * kRun);
    };
    // the run that k ends in: elements past k are zero whatever lies behind them (k is even: pairs are whole)
    auto load_x_tail = [&](Stage& st) {
        const int64_t k0 = (int64_t)a.full_runs * kRun;
        const int left = (int)(a.k - k0) - first;
#pragma unroll
        for (int i = 0; i < kRaw; ++i)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const int e = w * (4 / (int)sizeof(XT)), at = e + (kCompact ? i * kPiece : 0);
                uint32_t v = 0;
                if constexpr (kInt) {
                    const Any2* p = (const Any2*)(piece_of(i) + k0 + e);
                    if (at < left) v = p[0].a;
                    if (at + 2 < left) v |= (uint32_t)p[1].a << 16;
                } else {
                    if (at < left) v = ((const Any4<sizeof(XT)>*)(piece_of(i) + k0 + e))->a;
                }
                st.x[i][w] = v;
            }
    };

    // Operand slots of a wavefront: 16 bytes per (operand, step t, lane group q, column), the column rotated by the piece
    // so that the pieces of a column, written side by side, fall on different banks (and so do the columns of a read).
    uint32_t* const xs = lds + wave * kXWords;
    auto slot = [](int op, int t, int qq, int col) { return ((op * T + t) * 64 + qq * 16 + (col ^ (qq * T + t))) * 4; };
    auto put_x = [&](const Stage& st, auto split_one) {
        const int j = lane % kLanesPerCol;
#pragma unroll
        for (int i = 0; i < kRaw; ++i) {
            const int col = i * kColsPerLoad + lane / kLanesPerCol;
            if constexpr (sizeof(XT) == 4) {
                // half a slot: elements 4 (j & 1) .. + 3 of the 8 of step (j / 2) % 4
                Split s;
                split_one(st.x[i], s);
#pragma unroll
                for (int op = 0; op < 3; ++op) *(v2u*)&xs[slot(op, (j >> 1) & 3, j >> 3, col) + 2 * (j & 1)] = s.part[op];
            } else {
                *(v4u*)&xs[slot(0, j % T, j / T, col)] = st.x[i];
            }
        }
    };

    // The MFMAs add to the running sums themselves, except where a run's sum is scaled first, and for fp32: there a run's
    // three products are summed on their own and added once (adding them one by one to the running sum would round it
    // three times as often).
    constexpr bool kDirect = !kScaled && sizeof(XT) != 4;
    acc_t acc[R][kAcc];
    float sum[R];                                      // (scaled, compact) one column per lane
    acc_t total[R][kAcc];                              // int8: sums already shifted back
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int v = 0; v < kAcc; ++v) acc[r][v] = total[r][v] = acc_t{0, 0, 0, 0};
        sum[r] = 0.0f;
    }

    // a run's activations in operand order: in registers (compact) or in the wavefront's LDS buffer
    v4u x[kOps];
    auto operands = [&](const Stage& st, auto split_one) {
        if constexpr (kCompact && sizeof(XT) == 4) {
            Split s0, s1;
            split_one(st.x[0], s0);
            split_one(st.x[kRaw - 1], s1);
#pragma unroll
            for (int op = 0; op < kOps; ++op) x[op] = v4u{s0.part[op].x, s0.part[op].y, s1.part[op].x, s1.part[op].y};
        } else if constexpr (kCompact) {
            x[0] = st.x[0];
        } else {
            put_x(st, split_one);
        }
    };
    // ... times its weights, `unit` times added to the sums (fp32 only; 1 for the others)
    auto multiply = [&](const Stage& st, float unit, auto in_steps) {
        acc_t blk[R][kAcc];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            // (fp32: a step's operands are read together, ahead of its decoding; one by one, which the compiler does to save
            // registers, 4096 x 4096 x 8 takes 9.4 us instead of 7.5.  The widest instance has two wavefronts a SIMD and none
            // to spare: 14336 x 4096 x 16 15.4 one by one, 16.5 together.)
            constexpr bool kTogether = !kCompact && kOps > 1 && R * kCols4 < 16;
            if constexpr (kTogether) {
#pragma unroll
                for (int op = 0; op < kOps; ++op) x[op] = *(const v4u*)&xs[slot(op, t, q, n)];
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (decltype(in_steps)::value) __builtin_amdgcn_sched_barrier(0);
            v4u w[R];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if constexpr (F == kInt4) P::decode(st.codes[r], t, w[r]);
                else w[r] = convert<F, XT>(st.codes[2 * r + t / 2][2 * (t & 1)], st.codes[2 * r + t / 2][2 * (t & 1) + 1], a.times);
            }
#pragma unroll
            for (int op = kOps - 1; op >= 0; --op) {   // (the smallest part first)
                if constexpr (!kCompact && !kTogether) x[op] = *(const v4u*)&xs[slot(op, t, q, n)];
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    acc_t& to = kDirect ? acc[r][kCompact ? t : 0] : blk[r][kCompact ? t : 0];
                    const bool fresh = !kDirect && op == kOps - 1 && (kCompact || t == 0);
                    to = P::mma(x[op], w[r], fresh ? acc_t{0, 0, 0, 0} : to);
                }
            }
        }
        if constexpr (!kDirect) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                float s = kScaled ? __half2float(__ushort_as_half((uint16_t)(st.q[r / 2] >> (16 * (r & 1))))) : 1.0f;
                if constexpr (sizeof(XT) == 4) s *= unit;
                if constexpr (kCompact) {
                    sum[r] = fmaf(s, (blk[r][0][0] + blk[r][1 % kAcc][1]) + (blk[r][2 % kAcc][2] + blk[r][3 % kAcc][3]), sum[r]);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[r][0][i] = fmaf(s, blk[r][0][i], acc[r][0][i]);
                }
            }
        }
    };
    // fp32: the weight operands' factor goes in with each run, so that the sums are held at their own magnitude
    constexpr float kUnit = sizeof(XT) == 4 && F == kInt4 ? 16.0f : 1.0f;
    uint32_t lost = 0;                                 // bits that split has left out
    // (outside the loop the widest fp32 instance would run out of registers if the compiler did all steps at once)
    constexpr std::bool_constant<sizeof(XT) == 4 && kScaled && R * kCols4 >= 16> kInSteps;
    auto consume = [&](const Stage& st, auto in_steps) {
        if constexpr (sizeof(XT) == 4) {
            operands(st, [&](const v4u& v, Split& s) {
                split(v, s, lost);
                if constexpr (decltype(in_steps)::value) __builtin_amdgcn_sched_barrier(0);
            });
        } else {
            operands(st, 0);
        }
        multiply(st, kUnit, in_steps);
    };

    // Wavefront `wave` takes runs wave, wave + W, ... of the segment's full ones; the ragged one goes to the next in turn,
    // loaded first and added last.  The loop's loads are never skipped by a branch (a load that some paths leave out makes the
    // compiler wait for all of them): past the last run the codes come from past the end of the buffer, which reads no
    // memory, and the activations are those of the first run again.
    const int run0 = blockIdx.y * a.seg_runs, left_runs = a.full_runs - run0;
    const int here = left_runs <= 0 ? 0 : left_runs < a.seg_runs ? left_runs : a.seg_runs;
    const int mine = (here - wave + W - 1) / W;
    const bool tail = a.runs > a.full_runs && blockIdx.y == gridDim.y - 1 && wave == here % W;
    Stage tail_stage;
    if (tail) {
        load_codes_of(tail_stage, a.full_runs, true);
        load_x_tail(tail_stage);
    }
    auto shift_back = [&] {
        if constexpr (kInt) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int v = 0; v < kAcc; ++v)
#pragma unroll
                    for (int i = 0; i < 4; ++i) { total[r][v][i] += acc[r][v][i] >> 4; acc[r][v][i] = 0; }
        }
    };
    if (mine > 0) {
        Stage ring[D];
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const int run = run0 + wave + d * W;
            load_codes_of(ring[d], run, d < mine);
            load_x(ring[d], d < mine ? run : run0 + wave);
            __builtin_amdgcn_sched_barrier(0);
        }
        int it = 0;
        for (; it + D <= mine; it += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                consume(ring[d], std::false_type{});
                const int next = it + d + D;
                const int run = run0 + wave + next * W;
                load_codes_of(ring[d], run, next < mine);
                load_x(ring[d], next < mine ? run : run0 + wave);
                __builtin_amdgcn_sched_barrier(0);
            }
            // int8: 16 x the sum of a run stays under 2^21: shift back before 1024 runs can have overflowed
            if constexpr (kInt) if ((it / D & 63) == 63) shift_back();
        }
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (it + d < mine) consume(ring[d], kInSteps);
    }
    if (tail) consume(tail_stage, kInSteps);
    if constexpr (sizeof(XT) == 4) {
        // Infinities or NaNs (both have left NaNs in the sums): all over again.  Then what very small activations have lost.
        // Nothing of this is in the way otherwise: a look per run instead would cost 2 to 8 percent.
        float all = 0.0f;                              // (not a number if one of the sums is not)
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if constexpr (kCompact) all += sum[r];
            else all += (acc[r][0][0] + acc[r][0][1]) + (acc[r][0][2] + acc[r][0][3]);
        }
        const bool nan = (kCompact || 4 * q < kCols) && all != all;
        if (__builtin_amdgcn_ballot_w64(nan || (lost & 0xffffu) != 0)) {
            const bool again = __builtin_amdgcn_ballot_w64(nan) != 0;
            if (again) {
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    sum[r] = 0.0f;
                    acc[r][0] = acc_t{0, 0, 0, 0};
                }
            }
            const int last = run0 + wave + (mine - 1 + (tail ? 1 : 0)) * W;
            asm volatile("" : "+v"(lane));                 // (the addresses are worked out again rather than kept through the loop)
            locate();
            constexpr int kAtOnce = kCompact ? 4 : 1;      // runs requested together
            for (int pass = again ? 0 : 1; pass < 2; ++pass) {
#pragma unroll 1
                for (int run = run0 + wave; run <= last; run += kAtOnce * W) {
                    Stage st[kAtOnce];
#pragma unroll
                    for (int d = 0; d < kAtOnce; ++d) {
                        const int r = run + d * W <= last ? run + d * W : last;
                        load_codes_of(st[d], r, true);
                        if (r < a.full_runs) load_x(st[d], r);
                        else load_x_tail(st[d]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int d = 0; d < kAtOnce; ++d) {
                        if (run + d * W > last) break;
                        if (pass == 0) operands(st[d], [](const v4u& v, Split& s) { uint32_t l[4]; split_any(v, s, l); });
                        else operands(st[d], [](const v4u& v, Split& s) { split_lost(v, s); });
                        __builtin_amdgcn_sched_barrier(0);
                        multiply(st[d], pass == 0 ? kUnit : kUnit * kLostUnit, std::true_type{});
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        }
    }
    shift_back();

    // the wavefronts' sums, [wavefront][column][row]
    if constexpr (!kCompact) lds_barrier();            // (every wavefront has left its operands)
    auto bits = [](auto v) { uint32_t u; __builtin_memcpy(&u, &v, 4); return u; };
#pragma unroll
    for (int r = 0; r < R; ++r) {
        uint32_t* out = lds + wave * kCols * kPitch + r * 16 + n;
        if constexpr (kCompact && kInt) {
            out[(2 * q) * kPitch] = bits(total[r][0][0] + total[r][1 % kAcc][1]);
            out[(2 * q + 1) * kPitch] = bits(total[r][0][2] + total[r][1 % kAcc][3]);
        } else if constexpr (kCompact && !kDirect) {
            out[q * kPitch] = bits(sum[r]);
        } else if constexpr (kCompact) {
            out[q * kPitch] = bits((acc[r][0][0] + acc[r][1 % kAcc][1]) + (acc[r][2 % kAcc][2] + acc[r][3 % kAcc][3]));
        } else if (4 * q < kCols) {
#pragma unroll
            for (int i = 0; i < 4; ++i) out[(4 * q + i) * kPitch] = kInt ? bits(total[r][0][i]) : bits(acc[r][0][i]);
        }
    }
    __syncthreads();
    const int outs = kRows * ncols;
    for (int o = threadIdx.x; o < outs; o += W * 64) {
        const int c = o / kRows, row = o % kRows;
        const int64_t grow = (int64_t)rg * kRows + row;
        if (grow >= a.m) continue;
        using S = typename std::conditional<kInt, int, float>::type;
        S v[W];                                        // (in pairs: sixteen sums one after the other would round more than four did)
#pragma unroll
        for (int w = 0; w < W; ++w) __builtin_memcpy(&v[w], &lds[(w * kCols + c) * kPitch + row], 4);
#pragma unroll
        for (int step = 1; step < W; step *= 2)
#pragma unroll
            for (int w = 0; w < W; w += 2 * step) v[w] += v[w + step];
        S s = v[0];
        if (a.partials) {
            a.partials[((int64_t)blockIdx.y * a.b + col0 + c) * a.m_pad + grow] = bits(s);
            continue;
        }
        if constexpr (!kInt && !(F == kInt4 && !__is_same(XT, bf16_t))) s *= a.factor;
        ((YT*)a.Y)[(int64_t)(col0 + c) * a.ldy + grow] = to_output<YT, S>(s);
    }
}

// Tile kernel for int8 activations and a long k, up to 48 columns and, over a longer one, 64: the larger tiles of the kernel below have too little to do
// between its meetings there (8 steps of a microsecond and a half, 28672 x 4096 x 24: 15.6 us against 14.6).  A workgroup owns 64 R rows (four wavefronts of
// R row tiles) for all of k, or a segment of it, and up to 16 NT columns: two groups of four wavefronts take alternate runs, and the wavefronts
// of a group share the run's activations, staged in LDS in the streaming kernel's operand slots.  Activations and codes are requested five
// to six steps ahead (registers; three more steps in LDS): loads return in order, so a wait for activations is a wait for every code requested
// before them.  The operands of an MFMA step are read and decoded under the MFMAs of the one before it, also across the barrier.
template <typename XT, int R, int NT>
__global__ void __launch_bounds__(512)
matrix_small_tile_kernel(MatrixArgs a)
{
    using P = Policy<XT>;
    using acc_t = typename P::acc_t;
    using YT = typename P::out_t;
    constexpr int Wr = 4, Wk = 2;                      // wavefronts side by side in rows, groups of them along k
    constexpr int T = P::kFrags;
    constexpr int kPiece = 16 / (int)sizeof(XT);       // elements of a 16-byte piece
    constexpr int kLanesPerCol = kRun / kPiece, kColsPerLoad = 64 / kLanesPerCol;
    constexpr int kLoads = T * NT;                     // loads of a run's activations
    constexpr int kMine = (kLoads + Wr - 1) / Wr;      // of them a wavefront's
    constexpr int kCodesAhead = 6, kXAhead = 3, kBuffers = 3;
    constexpr int kRows = 16 * R * Wr;
    constexpr int kPitch = kRows + 4;
    constexpr int kXWords = Wk * kBuffers * kLoads * 256, kRedWords = 2 * Wk * 16 * kPitch;
    __shared__ __align__(16) uint32_t lds[kXWords > kRedWords ? kXWords : kRedWords];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave % Wr, g = wave / Wr;
    const int n = lane & 15, q = lane >> 4;
    // the column passes of one row group follow each other on one XCD: they stream the same codes
    const int unit = blockIdx.x / kXcds, pass = unit % a.passes;
    const int rg = unit / a.passes * kXcds + blockIdx.x % kXcds;
    if (rg >= a.row_groups) return;
    const int col0 = pass * NT * 16, ncols = a.b - col0 < NT * 16 ? a.b - col0 : NT * 16;
    // this segment's runs (the last one may be ragged)
    const int run0 = blockIdx.y * a.seg_runs;
    const int run1 = run0 + a.seg_runs < a.runs ? run0 + a.seg_runs : a.runs;

    constexpr uint32_t run_bytes = R * Wr * 1024u;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.codes + (int64_t)rg * a.runs * run_bytes), 0, (int)(a.runs * run_bytes), 0x00020000);
    struct Codes {
        v4u c[R];
        uint32_t unused;                               // (without it the compiler makes branches of the shifts below: 28672 x 4096 x 24 15.0 us, 14.6)
    };
    auto load_codes_of = [&](Codes& st, int run) {
        const bool ok = run < run1;
        const uint32_t off = (ok ? (uint32_t)run * run_bytes : kPastEnd) + wr * R * 1024u + lane * 16u;
#pragma unroll
        for (int r = 0; r < R; ++r)
            st.c[r] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(off + r * 1024u), 0, kAuxNt);
    };

    // Staging: load f = wr + i Wr of a run takes kColsPerLoad columns, consecutive lanes consecutive pieces.  The address
    // stops at the last whole piece of the column; what that moves is shifted back when the piece is put into LDS (only
    // from the run that k ends in on), zeros coming in: elements past k are zero whatever lies behind them.
    const XT* xcol[kMine];
    uint32_t xslot[kMine];
    const int xoff = lane % kLanesPerCol * kPiece;
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        int c = (wr + i * Wr) * kColsPerLoad + lane / kLanesPerCol;
        const int j = lane % kLanesPerCol;
        xslot[i] = ((c / 16 * T + j % T) * 64 + j / T * 16 + ((c & 15) ^ j)) * 4;
        c = c < ncols ? c : ncols - 1;
        xcol[i] = (const XT*)a.X + (int64_t)(col0 + c) * a.ldx;
    }
    const int last = (int)a.k - kPiece, whole = run1 < a.full_runs ? run1 : a.full_runs;
    auto load_x = [&](v4u (&x)[kMine], int run) {
        const int kk = run * kRun + xoff;
#pragma unroll
        for (int i = 0; i < kMine; ++i) x[i] = load_any16<sizeof(XT)>(xcol[i] + (kk < last ? kk : last));
    };
    auto put_x = [&](v4u (&x)[kMine], int run, int buf) {
        if (run >= whole) {
            const int sh = run < run1 ? run * kRun + xoff - last : kPiece;  // elements, even (past the segment: all)
            const int h = sh > 0 ? sh * (int)sizeof(XT) / 2 : 0;            // halfwords
#pragma unroll
            for (int i = 0; i < kMine; ++i) {
                v4u v = x[i];
                if (h & 1) v = v4u{v[0] >> 16 | v[1] << 16, v[1] >> 16 | v[2] << 16, v[2] >> 16 | v[3] << 16, v[3] >> 16};
                if (h & 2) v = v4u{v[1], v[2], v[3], 0};
                if (h & 4) v = v4u{v[2], v[3], 0, 0};
                if (h & ~7) v = v4u{0, 0, 0, 0};
                x[i] = v;
            }
        }
#pragma unroll
        for (int i = 0; i < kMine; ++i)
            if (kLoads % Wr == 0 || wr + i * Wr < kLoads) *(v4u*)&lds[(g * kBuffers + buf) * kLoads * 256 + xslot[i]] = x[i];
    };

    acc_t acc[R][NT];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) acc[r][nt] = acc_t{0, 0, 0, 0};
    auto read_x = [&](int buf, int t, int nt) {
        return *(const v4u*)&lds[((g * kBuffers + buf) * kLoads + nt * T + t) * 256 + q * 64 + (n ^ (q * T + t)) * 4];
    };
    auto decode = [&](v4u (&w)[R], const Codes& st, int t) {
#pragma unroll
        for (int r = 0; r < R; ++r) P::decode(st.c[r], t, w[r]);
    };

    // Step s: group g's run is run0 + g + s Wk (past the segment: codes from past the end, scale zero); all groups make the
    // same number of steps, rounded up to the unrolling.  At its start the activations of step s + 2 go to LDS and those of
    // s + 5 are requested, at its end the codes of s + 6.
    const int steps = (run1 - run0 + Wk - 1) / Wk;
    const auto run_of = [&](int s) { return run0 + g + s * Wk; };
    v4u xr[kXAhead][kMine], x[NT], w[2][R];
    Codes ring[kCodesAhead];
    load_codes_of(ring[0], run_of(0));
    load_x(xr[0], run_of(0));
    __builtin_amdgcn_sched_barrier(0);
    load_codes_of(ring[1], run_of(1));
    load_x(xr[1], run_of(1));
    __builtin_amdgcn_sched_barrier(0);
    load_codes_of(ring[2], run_of(2));
    load_x(xr[2], run_of(2));
    __builtin_amdgcn_sched_barrier(0);
    put_x(xr[0], run_of(0), 0);
    load_codes_of(ring[3], run_of(3));
    load_x(xr[0], run_of(3));
    __builtin_amdgcn_sched_barrier(0);
    put_x(xr[1], run_of(1), 1);
    load_codes_of(ring[4], run_of(4));
    load_x(xr[1], run_of(4));
    __builtin_amdgcn_sched_barrier(0);
    load_codes_of(ring[5], run_of(5));
    __builtin_amdgcn_sched_barrier(0);
    lds_barrier();
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) x[nt] = read_x(0, 0, nt);
    decode(w[0], ring[0], 0);
    for (int s = 0; s < steps; s += kCodesAhead) {
#pragma unroll
        for (int d = 0; d < kCodesAhead; ++d) {
            Codes& mine = ring[d];
            put_x(xr[(d + 2) % kXAhead], run_of(s + d + 2), (d + 2) % kBuffers);
            load_x(xr[(d + 2) % kXAhead], run_of(s + d + 2 + kXAhead));
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int now = (d * T + t) & 1, then = now ^ 1;
                const bool over = t + 1 == T;          // what is read ahead belongs to the next step
                decode(w[then], over ? ring[(d + 1) % kCodesAhead] : mine, over ? 0 : t + 1);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                    for (int r = 0; r < R; ++r) acc[r][nt] = P::mma(x[nt], w[now][r], acc[r][nt]);
                    x[nt] = read_x(over ? (d + 1) % kBuffers : d % kBuffers, over ? 0 : t + 1, nt);
                }
                constexpr int kDecode = 6;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                  // one MFMA
                        __builtin_amdgcn_sched_group_barrier(0x002, kDecode / NT + 1, 0);   // its share of the decoding
                    }
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                      // the tile's next operand
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            load_codes_of(mine, run_of(s + d + kCodesAhead));
            lds_barrier();
        }
    }
    // the groups' sums, a column tile at a time, [group][column][row] in alternating halves of the LDS
    auto bits = [](auto v) { uint32_t u; __builtin_memcpy(&u, &v, 4); return u; };
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        uint32_t* red = lds + (nt & 1) * Wk * 16 * kPitch;
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[r][nt][i] >>= 4;
                red[(g * 16 + 4 * q + i) * kPitch + (wr * R + r) * 16 + n] = bits(acc[r][nt][i]);
            }
        lds_barrier();
        for (int o = threadIdx.x; o < kRows * 16; o += Wr * Wk * 64) {
            const int c = nt * 16 + o / kRows, row = o % kRows;
            const int64_t grow = (int64_t)rg * kRows + row;
            if (grow >= a.m || c >= ncols) continue;
            int sum = 0;
#pragma unroll
            for (int k = 0; k < Wk; ++k) {
                int v;
                __builtin_memcpy(&v, &red[(k * 16 + c % 16) * kPitch + row], 4);
                sum += v;
            }
            if (a.partials) {
                a.partials[((int64_t)blockIdx.y * a.b + col0 + c) * a.m_pad + grow] = bits(sum);
                continue;
            }
            ((YT*)a.Y)[(int64_t)(col0 + c) * a.ldy + grow] = sum;
        }
    }
}

// Tile kernel, more columns than the streaming kernel holds.  A workgroup owns 64 R rows for all of k, or a segment of it, and up
// to 32 NT columns.  Four pairs of wavefronts take alternate runs of 128 columns of k; each wavefront of a pair has R tiles of 32 rows, and the
// pair shares the run's activations, staged in LDS.
//
// What bounds it, and what the shape is for (49152 x 12288 x 64 fp16, 28672 x 8192 x 64 bf16 with scales):
//   * Issue of vector and matrix instructions, and power.  A SIMD issues a matrix instruction in 8 clocks and a vector instruction in 4.7, whichever
//     of its two wavefronts they come from: products of 32 x 32 need half as many as products of 16 x 16.  With them 2.3 (4.3 with scales) vector
//     instructions per 16 x 16 x 32 products fit beside the matrix cores' own 16 clocks.  The clock falls to 1.5 GHz under 49152 x 12288 x 64;
//     with activations of zero it takes 65 us.
//   * LDS: two wavefronts read a run's activations, where four did in tiles of 16 rows.
//   * Vector memory: 112 KiB of codes and activations a step and compute unit, 1800 of its 4300 clocks.  Activations go straight to the LDS (through
//     registers 91 us instead of 79), and no wavefront asks for much at once: the next step's activations in the first half of a step, then
//     the codes of the step after it, which come from memory and have a step more to arrive.
//   * One meeting of the wavefronts a step, behind it.  Ahead of the last products of a step: level.
// Measured, us: 49152 x 12288 x 64 fp16 77 to 86 on different cards = 0.9 to 1.0 Pflop/s (tiles of 16 rows with activations through registers 87 to 93), 28672 x 8192 x 64
// bf16 with scales 41 to 45 (52 to 59), 16384 x 4096 x 64 15.6 to 16.2 (21), 14336 x 4096 x 32 12.6 (14.3), 28672 x 4096 x 64 int8 18.6 (20.9), 28672 x 8192 x 64 fp16 with
// E4M3 codes 48 (passes of the streaming kernel 161), 25856 x 6144 x 24 29.5 (53).  Level or slower: wavefronts of
// different priority, an interleaving of products and decoding laid down by hand.
// 32 x 32 products, sixteen (int8: 32) columns of k at a time
template <typename XT> struct Big {
    using acc_t = v16f;
    static constexpr int kSteps = 8, kVecSteps = 4;    // per run; per 16-byte load of codes
    static __device__ __forceinline__ v16f mma(const v4u& x, const v4u& w, const v16f& c)
    {
        if constexpr (__is_same(XT, __half))
            return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, x), __builtin_bit_cast(v8h, w), c, 0, 0, 0);
        else
            return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8bf, x), __builtin_bit_cast(v8bf, w), c, 0, 0, 0);
    }
};
template <> struct Big<int8_t> {
    using acc_t = v16i;
    static constexpr int kSteps = 4, kVecSteps = 2;
    static __device__ __forceinline__ v16i mma(const v4u& x, const v4u& w, const v16i& c)
    {
        return __builtin_amdgcn_mfma_i32_32x32x32_i8(__builtin_bit_cast(v4i, x), __builtin_bit_cast(v4i, w), c, 0, 0, 0);
    }
};

template <typename XT, int F, int R, int NT, bool kScaled, bool kDirect>
__global__ void __launch_bounds__(512)
matrix_tile_kernel(MatrixArgs a)
{
    using P = Policy<XT>;
    using G = Big<XT>;
    using acc_t = typename G::acc_t;
    using YT = typename P::out_t;
    static_assert(sizeof(XT) != 4 && !(kScaled && R > 2));
    constexpr bool kInt = sizeof(XT) == 1;
    constexpr int Wr = kTileRowWaves, Wk = 8 / Wr;
    constexpr int T = G::kSteps;
    constexpr int kVecs = F == kInt4 ? 2 : 4;          // loads of codes per row tile and run
    constexpr int kPiece = 16 / (int)sizeof(XT);       // elements of a 16-byte piece
    constexpr int kPieces = kRun / kPiece;             // pieces of a column's run
    constexpr int kColsPerLoad = 64 / kPieces;         // a wavefront's load: 1 KiB of LDS
    constexpr int kMine = 32 * NT / kColsPerLoad / Wr; // of a run's loads a wavefront's
    constexpr uint32_t kTileBytes = 32 * NT * kRun * sizeof(XT), kStageBytes = Wk * kTileBytes;
    constexpr int kRows = 32 * R * Wr;
    // the final sum: column tiles at a time, and words from row to row (16 rows' pieces of 16 bytes fall on different banks)
    constexpr int kAtOnce = R < 3 ? NT : 1, kPitch = 32 * kAtOnce + 4;
    constexpr int Rp = R == 3 ? 4 : R;                 // scales per lane and block, padded to a power of two
    constexpr uint32_t kRedBytes = Wk * kRows * kPitch * 4;
    __shared__ __align__(1024) uint8_t lds[2 * kStageBytes > kRedBytes ? 2 * kStageBytes : kRedBytes];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wr = wave % Wr, g = wave / Wr;
    const int n = lane & 31, h = lane >> 5;
    // the column passes of one row group follow each other on one XCD: they stream the same codes
    const int unit = blockIdx.x / kXcds, pass = unit % a.passes;
    const int rg = unit / a.passes * kXcds + blockIdx.x % kXcds;
    if (rg >= a.row_groups) return;
    const int col0 = pass * NT * 32, ncols = a.b - col0 < NT * 32 ? a.b - col0 : NT * 32;
    // what the end needs is fetched now: there the trip of the scalar loads would be in the way
    YT* Y = (YT*)a.Y;
    uint32_t* partials = a.partials;
    int64_t ldy = a.ldy, m = a.m;
    float factor = a.factor;
    const float times = a.times;
    asm volatile("" : "+s"(Y), "+s"(partials), "+s"(ldy), "+s"(m), "+s"(factor));
    // this segment's runs; a ragged one (the last of k) goes first, so that what it takes is part of the start
    const int run0 = blockIdx.y * a.seg_runs;
    const int run1 = run0 + a.seg_runs < a.runs ? run0 + a.seg_runs : a.runs;
    const int nruns = run1 - run0, ragged = run1 > a.full_runs ? 1 : 0;
    const int steps = (nruns + Wk - 1) / Wk;

    constexpr uint32_t run_bytes = R * Wr * kVecs * 1024u;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.codes + (int64_t)rg * a.runs * run_bytes), 0, (int)(a.runs * run_bytes), 0x00020000);
    constexpr int kScaleRow = Wr * 32 * Rp;
    const __amdgpu_buffer_rsrc_t srsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(a.scales + (int64_t)rg * a.nblocks * kScaleRow), 0, kScaled ? (int)(a.nblocks * kScaleRow * 2) : 0, 0x00020000);

    // Activations.  Load i of a run takes kColsPerLoad columns, a lane 16 bytes, which go to 16 bytes of LDS in the lanes' order; which
    // piece of its column a lane takes is turned by the column, so that the lanes that read one piece of 16 columns find them on
    // different banks while every load still covers whole runs of columns.
    const auto turn = [](int col) { return kInt ? (col >> 1) & 7 : col & 15; };
    const uint8_t* const xbase = (const uint8_t*)((const XT*)a.X + (int64_t)col0 * a.ldx);
    using off_t = typename std::conditional<kDirect, uint32_t, int64_t>::type;   // (direct: the host has seen that 32 bits are enough)
    off_t xoff[kMine];                                 // bytes from xbase, at the first run
    int xpiece[kMine];
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        const int slot = (wr + i * Wr) * kColsPerLoad + lane / kPieces;
        xpiece[i] = (lane % kPieces ^ turn(slot)) * kPiece;
        xoff[i] = (off_t)((slot < ncols ? slot : ncols - 1) * a.ldx * (int64_t)sizeof(XT)) + xpiece[i] * (int)sizeof(XT);
    }
    const uint64_t xaddr = (uint64_t)xbase;
    const v4i xrsrc = {(int)(uint32_t)xaddr, (int)((uint32_t)(xaddr >> 32) & 0xffffu), (int)0x7fffffff, 0x00020000};
    uint8_t* const mine = lds + g * kTileBytes;

    struct Codes {
        v4u c[R][kVecs];
        uint32_t q[1];
    };
    v4u xr[kDirect ? 1 : kMine];
    const auto run_at = [&](int i) { return ragged ? (i == 0 ? run1 - 1 : run0 + i - 1) : run0 + i; };
    // (a step past the last run: the codes come from past the end of the buffer, the activations are those of the first run again)
    const auto load_code = [&](Codes& st, bool ok, int run, int j) {
        const uint32_t off = (ok ? (uint32_t)run * run_bytes : kPastEnd) + wr * R * kVecs * 1024u + lane * 16u;
        st.c[j / kVecs][j % kVecs] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(off + j * 1024u), 0, kAuxNt);
    };
    const auto load_scales = [&](Codes& st, bool ok, int run) {
        if constexpr (kScaled) {
            const uint32_t so = (ok ? fast_div((uint32_t)run, a.div_block) * (uint32_t)(kScaleRow * 2) : kPastEnd) + (wr * 32 + n) * (uint32_t)(Rp * 2);
            if constexpr (Rp == 2) st.q[0] = __builtin_amdgcn_raw_buffer_load_b32(srsrc, (int)so, 0, 0);
            else st.q[0] = (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(srsrc, (int)so, 0, 0);
        }
    };
    const auto load_x = [&](uint32_t buf, int run, int j) {
        if constexpr (kDirect) {
            const uint32_t to = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)mine + buf + (wr + j * Wr) * 1024u;
            // (the wait states are those behind a vector instruction that writes a scalar operand, which the compiler does not count into asm.  What is
            // written is the LDS: `arrive`, which clobbers memory, stands between this load and every read of what it brings, and between the reads
            // of what was there and this load.  A clobber here too costs 2 percent at 14336 x 4096 x 32, 12.1 us and 12.4: the addresses are worked out later.)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                         :: "s"(to), "v"(xoff[j]), "s"(xrsrc), "s"(run * (int)(kRun * sizeof(XT))) : "m0");
        } else {
            xr[j] = load_any16<sizeof(XT)>(xbase + xoff[j] + (int64_t)run * (int)(kRun * sizeof(XT)));
        }
    };
    const auto put = [&](int i, uint32_t buf, const v4u& v) { *(v4u*)&mine[buf + (wr + i * Wr) * 1024 + lane * 16] = v; };
    // The ragged run: the address stops at the last whole piece of the column, what that moves is shifted back, zeros coming in
    // (elements past k are zero whatever lies behind them).
    const auto stage_ragged = [&] {
        const int last = (int)a.k - kPiece;
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const int kk = a.full_runs * kRun + xpiece[i], at = kk < last ? kk : last;
            v4u v = load_any16<sizeof(XT)>(xbase + xoff[i] + (int64_t)(at - xpiece[i]) * (int)sizeof(XT));
            const int h2 = (kk - at) * (int)sizeof(XT) / 2;   // halfwords
            if (h2 & 1) v = v4u{v[0] >> 16 | v[1] << 16, v[1] >> 16 | v[2] << 16, v[2] >> 16 | v[3] << 16, v[3] >> 16};
            if (h2 & 2) v = v4u{v[1], v[2], v[3], 0};
            if (h2 & 4) v = v4u{v[2], v[3], 0, 0};
            if (h2 & ~7) v = v4u{0, 0, 0, 0};
            put(i, 0, v);
        }
    };
    // the first step's, requested at once
    const auto request = [&](Codes& st) {
        if (g >= nruns) return;
        const int run = run_at(g);
        if (run < a.full_runs) {
#pragma unroll
            for (int j = 0; j < kMine; ++j) load_x(0, run, j);
            if constexpr (!kDirect) {
#pragma unroll
                for (int j = 0; j < kMine; ++j) put(j, 0, xr[j]);
            }
        } else {
            stage_ragged();
        }
#pragma unroll
        for (int j = 0; j < kVecs * R; ++j) load_code(st, true, run, j);
        load_scales(st, true, run);
    };
    // The next step's activations are in LDS for every wavefront when this returns, its codes in registers; the codes of the one after it are
    // still on their way: `later` loads, the last that were asked for.
    const auto arrive = [&](auto later) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"(decltype(later)::value) : "memory");
    };

    acc_t acc[R][NT];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[r][nt][i] = 0;
    const uint32_t xread = g * kTileBytes + (uint32_t)n * (kPieces * 16u) + (uint32_t)((h * T) ^ turn(n)) * 16u;
    // A step, and the requests behind it, spread over it: asked for at once they queue up in front of the vector memory unit, and the
    // wavefront with them.  The activations of the next step go first (they come from the L2), then the codes of the one after it, which
    // have a step more to arrive.
    v4u w[2][R], x[2][NT];
    constexpr int kHalf = T / 2;
    constexpr int kLater = kVecs * R + (kScaled ? 1 : 0);
    const auto decode = [&](v4u& to, const v4u (&c)[kVecs], int t) {
        if constexpr (F == kInt4) P::decode(c[t / G::kVecSteps], t % G::kVecSteps, to);
        else to = convert<F, XT>(c[t / 2][2 * (t & 1)], c[t / 2][2 * (t & 1) + 1], times);
    };
    const auto compute = [&](const Codes& st, const Codes& next, Codes& later, int s, uint32_t buf) {
        const bool ok1 = (s + 1) * Wk + g < nruns, ok2 = (s + 2) * Wk + g < nruns;
        const int run1 = ok1 ? run_at((s + 1) * Wk + g) : 0, run2 = ok2 ? run_at((s + 2) * Wk + g) : 0;
        acc_t blk[kScaled ? R : 1][kScaled ? NT : 1];
        const uint32_t from = xread + buf;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) x[0][nt] = *(const v4u*)&lds[from + nt * 32 * kPieces * 16];
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int now = t & 1, then = now ^ 1;
            if (t < kHalf) {
#pragma unroll
                for (int j = t * kMine / kHalf; j < (t + 1) * kMine / kHalf; ++j) load_x(buf ^ kStageBytes, run1, j);
            } else {
#pragma unroll
                for (int j = (t - kHalf) * kVecs * R / kHalf; j < (t + 1 - kHalf) * kVecs * R / kHalf; ++j) load_code(later, ok2, run2, j);
                if (t == kHalf) load_scales(later, ok2, run2);
            }
            if (t + 1 < T) {
                const uint32_t at = from ^ (uint32_t)((t + 1) * 16);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) x[then][nt] = *(const v4u*)&lds[at + nt * 32 * kPieces * 16];
            }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (t + 1 < T) decode(w[then][r], st.c[r], t + 1);
                else decode(w[then][r], next.c[r], 0);
            }
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    if constexpr (kScaled) {
                        if (t == 0)
#pragma unroll
                            for (int i = 0; i < 16; ++i) blk[r][nt][i] = 0;
                        blk[r][nt] = G::mma(x[now][nt], w[now][r], blk[r][nt]);
                    } else {
                        acc[r][nt] = G::mma(x[now][nt], w[now][r], acc[r][nt]);
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (kScaled) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float q = __half2float(__ushort_as_half((uint16_t)(st.q[r / 2] >> (16 * (r & 1)))));
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[r][nt][i] = fmaf(q, blk[r][nt][i], acc[r][nt][i]);
                    asm volatile("" : "+v"(acc[r][nt]));   // (here and now: the compiler would keep all steps' sums until the end of the loop)
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    Codes ring[3];
    request(ring[0]);
    {
        const bool ok = Wk + g < nruns;
        const int run = ok ? run_at(Wk + g) : 0;
#pragma unroll
        for (int j = 0; j < kVecs * R; ++j) load_code(ring[1], ok, run, j);
        load_scales(ring[1], ok, run);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) decode(w[0][r], ring[0].c[r], 0);
    arrive(std::integral_constant<int, kLater>{});
    uint32_t buf = 0;
    for (int s = 0; s < steps; s += 3) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            if (s + d < steps) {
                if ((s + d) * Wk + g < nruns) {
                    compute(ring[d], ring[(d + 1) % 3], ring[(d + 2) % 3], s + d, buf);
                    if constexpr (!kDirect) {
#pragma unroll
                        for (int j = 0; j < kMine; ++j) put(j, buf ^ kStageBytes, xr[j]);
                    }
                }
                arrive(std::integral_constant<int, kLater>{});
                buf ^= kStageBytes;
            }
        }
    }
    arrive(std::integral_constant<int, 0>{});
    // the pairs' sums, [pair][row][column], four columns of a row at a time
    auto bits = [](auto v) { uint32_t u; __builtin_memcpy(&u, &v, 4); return u; };
    uint32_t* const red = (uint32_t*)lds;
    using S = typename std::conditional<kInt, int, float>::type;
#pragma unroll
    for (int n0 = 0; n0 < NT; n0 += kAtOnce) {
        if (n0) lds_barrier();
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int nt = n0; nt < n0 + kAtOnce; ++nt)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    v4u v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if constexpr (kInt) acc[r][nt][4 * i + e] >>= 4;
                        v[e] = bits(acc[r][nt][4 * i + e]);
                    }
                    *(v4u*)&red[(g * kRows + (wr * R + r) * 32 + n) * kPitch + (nt - n0) * 32 + 8 * i + 4 * h] = v;
                }
        lds_barrier();
#pragma unroll
        for (int o = 0; o < R * kAtOnce; ++o) {
            const int at = o * 512 + threadIdx.x, row = at % kRows, c = at / kRows * 4;
            const int64_t grow = (int64_t)rg * kRows + row;
            S sum[4] = {0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < Wk; ++k) {
                S v[4];
                __builtin_memcpy(v, &red[(k * kRows + row) * kPitch + c], 16);
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[e] += v[e];
            }
            const int col = n0 * 32 + c, left = grow < m ? ncols - col : 0;
            if (partials) {
                uint32_t* const to = partials + ((int64_t)blockIdx.y * a.b + col0 + col) * a.m_pad + grow;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e < left) to[e * a.m_pad] = bits(sum[e]);
            } else {
                YT* const to = Y + (int64_t)(col0 + col) * ldy + grow;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    if constexpr (!kInt && !(F == kInt4 && __is_same(XT, __half))) sum[e] *= factor;
                    if (e < left) to[e * ldy] = to_output<YT, S>(sum[e]);
                }
            }
        }
    }
}

// The segments' sums, in order.  Bound by the trip to memory of a handful of loads: 2.6 us for 256 rows of three columns, 4.6 to
// 6 for 64 columns of 4096 to 12288 rows.  What a cut has to win back is more, the writing of the sums and the launch with it: see
// segments_of in matrix_choose_shape.
template <typename XT>
__global__ void __launch_bounds__(256)
matrix_reduce_kernel(MatrixArgs a, int segments)
{
    using YT = typename Policy<XT>::out_t;
    using S = typename std::conditional<sizeof(XT) == 1, int, float>::type;
    const int64_t row = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (row >= a.m) return;
    const int c = blockIdx.y;
    S s = 0;
    for (int seg = 0; seg < segments; ++seg) {
        S v;
        __builtin_memcpy(&v, &a.partials[((int64_t)seg * a.b + c) * a.m_pad + row], 4);
        s += v;
    }
    if constexpr (sizeof(XT) != 1) s *= a.factor;
    ((YT*)a.Y)[(int64_t)c * a.ldy + row] = to_output<YT, S>(s);
}

// Row-major codes -> the order above (inverse: back again).  Once per plan; 32 MiB in 65 us, bound by the row-major side,
// where neighbouring lanes are a row apart.
template <bool kInverse, bool kTall>
__global__ void __launch_bounds__(256)
matrix_repack_kernel(uint8_t* __restrict__ rows, uint8_t* __restrict__ tiled, int64_t m, int64_t k, int64_t runs, int R,
                     int enc, int64_t dwords)
{
    const int64_t kbytes = k / 2;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dwords; i += (int64_t)gridDim.x * blockDim.x) {
        const int w = (int)(i & 3), lane = (int)(i >> 2) & 63;
        const int64_t tile = i >> (kTall ? 9 : 8);          // (row group, run, r)
        const int r = (int)(tile % R);
        const int64_t rest = tile / R;
        const int64_t run = rest % runs, rg = rest / runs;
        const int64_t row = kTall ? (rg * R + r) * 32 + (lane & 31) : (rg * R + r) * 16 + (lane & 15);
        const int64_t byte0 = (run * kRun + (kTall ? 64 * (lane >> 5) + 32 * ((int)(i >> 8) & 1) : 32 * (lane >> 4)) + 8 * w) / 2;
        uint8_t* src = rows + row * kbytes + byte0;
        uint32_t v = kInverse ? ((const uint32_t*)tiled)[i] : 0;
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const bool ok = row < m && byte0 + e / 2 < kbytes;
            const int p0 = 4 * nibble_of(enc, e), p1 = 4 * nibble_of(enc, e + 1);
            if constexpr (kInverse) {
                if (ok) src[e / 2] = (uint8_t)(stored_code(enc, (v >> p0) & 15u) | stored_code(enc, (v >> p1) & 15u) << 4);
            } else {
                const uint32_t byte = ok ? src[e / 2] : 0u;
                v |= stored_code(enc, byte & 15u) << p0 | stored_code(enc, byte >> 4) << p1;
            }
        }
        if constexpr (!kInverse) ((uint32_t*)tiled)[i] = v;
    }
}

// Row-major 8-bit codes -> the order above; a pattern that the format does not read as its value is replaced by one it does.
struct Remap { uint8_t to[256]; };
template <bool kTall>
__global__ void __launch_bounds__(256)
matrix_repack8_kernel(const uint8_t* __restrict__ rows, uint8_t* __restrict__ tiled, int64_t m, int64_t k, int64_t runs,
                      int R, Remap remap, int64_t dwords)
{
    __shared__ uint8_t to[256];
    to[threadIdx.x] = remap.to[threadIdx.x];
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < dwords; i += (int64_t)gridDim.x * blockDim.x) {
        const int w = (int)(i & 3), lane = (int)(i >> 2) & 63, part = (int)(i >> 8) & (kTall ? 3 : 1);
        const int64_t tile = i >> (kTall ? 10 : 9);         // (row group, run, r)
        const int64_t run = tile / R % runs, rg = tile / R / runs;
        const int64_t row = kTall ? (rg * R + tile % R) * 32 + (lane & 31) : (rg * R + tile % R) * 16 + (lane & 15);
        const int64_t col = run * kRun + (kTall ? 64 * (lane >> 5) : 32 * (lane >> 4)) + 16 * part + 4 * w;
        uint32_t v = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (row < m && col + e < k) v |= (uint32_t)to[rows[row * k + col + e]] << (8 * e);
        ((uint32_t*)tiled)[i] = v;
    }
}

// scales [m][nblocks] -> [row group][scale block][row wavefront][n][its row tiles, padded to Rp]; rows past m get zero
template <int kHeight>
__global__ void __launch_bounds__(256)
matrix_repack_scales_kernel(const __half* __restrict__ scales, __half* __restrict__ ordered, int64_t m, int64_t nblocks,
                            int R, int Wr, int Rp, int64_t total)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int r = (int)(i % Rp), n = (int)(i / Rp) % kHeight, wr = (int)(i / (kHeight * Rp) % Wr);
        const int64_t rest = i / (kHeight * Rp * Wr);
        const int64_t block = rest % nblocks, rg = rest / nblocks;
        const int64_t row = ((rg * Wr + wr) * R + r) * kHeight + n;
        ordered[i] = r < R && row < m ? scales[row * nblocks + block] : __float2half(0.0f);
    }
}

template <typename XT> int reduce_segments(const Plan& p, const MatrixArgs& a, hipStream_t s)
{
    if (p.mx_segments > 1) {
        hipLaunchKernelGGL(matrix_reduce_kernel<XT>, dim3((unsigned)((a.m + 255) / 256), (unsigned)a.b), dim3(256), 0, s, a,
                           p.mx_segments);
        MSGEMM_HIP_TRY(hipGetLastError());
    }
    return MSGEMM_OK;
}

template <typename XT, int R, int kCols4, int W, int D, int F>
int launch_stream(const Plan& p, const MatrixArgs& a, hipStream_t s)
{
    const dim3 grid((unsigned)p.row_blocks, (unsigned)p.mx_segments, (unsigned)a.passes), block(W * 64);
    if (sizeof(XT) != 1 && a.scales)
        hipLaunchKernelGGL((matrix_stream_kernel<XT, R, kCols4, W, D, sizeof(XT) != 1, F>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((matrix_stream_kernel<XT, R, kCols4, W, D, false, F>), grid, block, 0, s, a);
    MSGEMM_HIP_TRY(hipGetLastError());
    return reduce_segments<XT>(p, a, s);
}

template <typename XT, int F, int R, int NT>
int launch_tile(const Plan& p, const MatrixArgs& a, hipStream_t s)
{
    const dim3 grid((unsigned)(kXcds * a.passes * ((a.row_groups + kXcds - 1) / kXcds)), (unsigned)p.mx_segments);
    // (scaled sums are held twice)
    constexpr bool kCanScale = sizeof(XT) != 1 && (F == kInt4 ? R < 3 : R * NT < 4);
    if (sizeof(XT) != 1 && !kCanScale && a.scales) return MSGEMM_ERR_UNSUPPORTED;
    // straight into the LDS (at any alignment) where 32 bits reach every piece
    const bool direct = (32 * NT + 1) * a.ldx * (int64_t)sizeof(XT) < (1ll << 31);
    const bool scaled = kCanScale && a.scales;
    if (scaled && direct) hipLaunchKernelGGL((matrix_tile_kernel<XT, F, R, NT, kCanScale, true>), grid, dim3(512), 0, s, a);
    else if (scaled) hipLaunchKernelGGL((matrix_tile_kernel<XT, F, R, NT, kCanScale, false>), grid, dim3(512), 0, s, a);
    else if (direct) hipLaunchKernelGGL((matrix_tile_kernel<XT, F, R, NT, false, true>), grid, dim3(512), 0, s, a);
    else hipLaunchKernelGGL((matrix_tile_kernel<XT, F, R, NT, false, false>), grid, dim3(512), 0, s, a);
    MSGEMM_HIP_TRY(hipGetLastError());
    return reduce_segments<XT>(p, a, s);
}

template <typename XT>
int launch_tile_for_type(const Plan& p, const MatrixArgs& a, hipStream_t s)
{
#define MSGEMM_CASE(RR, NN) \
    if (p.mx_r == RR && p.mx_cols == 2 * NN) return launch_tile<XT, kInt4, RR, NN>(p, a, s);
    MSGEMM_CASE(1, 1) MSGEMM_CASE(2, 1) MSGEMM_CASE(3, 1)
    MSGEMM_CASE(1, 2) MSGEMM_CASE(2, 2) MSGEMM_CASE(3, 2)
#undef MSGEMM_CASE
    return MSGEMM_ERR_UNSUPPORTED;
}

template <int R, int NT>
int launch_small(const Plan& p, const MatrixArgs& a, hipStream_t s)
{
    const dim3 grid((unsigned)(kXcds * a.passes * ((a.row_groups + kXcds - 1) / kXcds)), (unsigned)p.mx_segments);
    hipLaunchKernelGGL((matrix_small_tile_kernel<int8_t, R, NT>), grid, dim3(512), 0, s, a);
    MSGEMM_HIP_TRY(hipGetLastError());
    return reduce_segments<int8_t>(p, a, s);
}

int launch_small_tile(const Plan& p, const MatrixArgs& a, hipStream_t s)
{
#define MSGEMM_CASE(RR, NN) \
    if (p.mx_r == RR && p.mx_cols == NN) return launch_small<RR, NN>(p, a, s);
    MSGEMM_CASE(1, 2) MSGEMM_CASE(2, 2) MSGEMM_CASE(3, 2) MSGEMM_CASE(1, 3) MSGEMM_CASE(2, 3) MSGEMM_CASE(3, 3)
    MSGEMM_CASE(1, 4) MSGEMM_CASE(2, 4) MSGEMM_CASE(3, 4)
#undef MSGEMM_CASE
    return MSGEMM_ERR_UNSUPPORTED;
}

template <typename XT, int F>
int launch_tile_for_codes8(const Plan& p, const MatrixArgs& a, hipStream_t s)
{
#define MSGEMM_CASE(RR, NN) \
    if (p.mx_r == RR && p.mx_cols == 2 * NN) return launch_tile<XT, F, RR, NN>(p, a, s);
    MSGEMM_CASE(1, 1) MSGEMM_CASE(2, 1) MSGEMM_CASE(1, 2) MSGEMM_CASE(2, 2)
#undef MSGEMM_CASE
    return MSGEMM_ERR_UNSUPPORTED;
}

template <typename XT>
int launch_for_type(const Plan& p, const MatrixArgs& a, hipStream_t s)
{
#define MSGEMM_CASE(RR, CC, WW, DD) \
    if (p.mx_r == RR && p.mx_cols == CC && p.mx_waves == WW && p.mx_depth == DD) return launch_stream<XT, RR, CC, WW, DD, kInt4>(p, a, s);
    MSGEMM_CASE(4, 0, 4, 2)
    MSGEMM_CASE(2, 0, 4, 4)
    MSGEMM_CASE(1, 0, 4, 2) MSGEMM_CASE(1, 0, 4, 4) MSGEMM_CASE(1, 0, 16, 2)
    if constexpr (sizeof(XT) != 1) {
        MSGEMM_CASE(2, 0, 4, 2)
    }
    if constexpr (sizeof(XT) != 4) {
        MSGEMM_CASE(2, 0, 8, 2) MSGEMM_CASE(1, 0, 4, 8) MSGEMM_CASE(1, 0, 8, 4)
    } else {
        MSGEMM_CASE(4, 2, 4, 2) MSGEMM_CASE(1, 2, 4, 2)
        MSGEMM_CASE(2, 4, 4, 2) MSGEMM_CASE(1, 4, 4, 2)
    }
    if constexpr (sizeof(XT) != 1) {  // (int8: the compact form holds eight columns)
        MSGEMM_CASE(4, 2, 8, 2) MSGEMM_CASE(2, 2, 8, 2) MSGEMM_CASE(1, 2, 8, 2) MSGEMM_CASE(2, 2, 4, 2)
    }
    if constexpr (__is_same(XT, __half)) {
        MSGEMM_CASE(2, 4, 4, 4)
    }
    if constexpr (sizeof(XT) == 1) {
        MSGEMM_CASE(2, 4, 4, 2) MSGEMM_CASE(2, 4, 4, 4) MSGEMM_CASE(1, 4, 4, 4)
    }
    MSGEMM_CASE(4, 4, 8, 2) MSGEMM_CASE(4, 4, 4, 2) MSGEMM_CASE(2, 4, 8, 2) MSGEMM_CASE(1, 4, 8, 2)
#undef MSGEMM_CASE
    return MSGEMM_ERR_UNSUPPORTED;
}

template <typename XT, int F>
int launch_for_codes8(const Plan& p, const MatrixArgs& a, hipStream_t s)
{
#define MSGEMM_CASE(RR, CC, DD) \
    if (p.mx_r == RR && p.mx_cols == CC && p.mx_depth == DD) return launch_stream<XT, RR, CC, 4, DD, F>(p, a, s);
    MSGEMM_CASE(2, 0, 4)
    MSGEMM_CASE(1, 0, 4)
    MSGEMM_CASE(2, 2, 2)
    // (fp32: rings of four take all registers of a SIMD for one wavefront; 4096 x 4096 x 8 8.4 us, in twos 7.5, 20000 x 512 x 8 15.4 / 7.4)
    constexpr int kDeep = sizeof(XT) == 4 ? 2 : 4;
    MSGEMM_CASE(1, 2, kDeep)
    MSGEMM_CASE(2, 4, 2)
    MSGEMM_CASE(1, 4, 2)
#undef MSGEMM_CASE
    return MSGEMM_ERR_UNSUPPORTED;
}

template <typename XT> int launch_for_format(const Plan& p, const MatrixArgs& a, hipStream_t s)
{
    if constexpr (sizeof(XT) == 2) {
        if (p.mx_tall) return p.mx_format == kE4M3 ? launch_tile_for_codes8<XT, kE4M3>(p, a, s) : launch_tile_for_codes8<XT, kE5M2>(p, a, s);
    }
    return p.mx_format == kE4M3 ? launch_for_codes8<XT, kE4M3>(p, a, s) : launch_for_codes8<XT, kE5M2>(p, a, s);
}

// Finite value of a pattern of a format (OCP 8-bit formats: bias 7 and 15; E4M3 has no infinities and one NaN a sign).
bool format_value(int format, int pattern, double& v)
{
    const int mb = format == kE4M3 ? 3 : 2, bias = format == kE4M3 ? 7 : 15;
    const int e = (pattern & 0x7f) >> mb, f = pattern & ((1 << mb) - 1);
    if (format == kE4M3 ? (pattern & 0x7f) == 0x7f : e == 31) return false;
    v = e == 0 ? ldexp((double)f, 1 - bias - mb) : ldexp(1.0 + ldexp((double)f, -mb), e - bias);
    if (pattern & 0x80) v = -v;
    return true;
}

}  // namespace

// Whether a map of 256 values is one of the formats the device converts, times a power of two; a pattern that stands for
// no number in the format must have a value that another pattern has.
void matrix_find_format(Plan& p, const float* values)
{
    p.mx_format = kInt4;
    for (int format : {kE4M3, kE5M2}) {
        const float one = values[format == kE4M3 ? 0x38 : 0x3c];
        int exponent = 0;
        if (!(one > 0.0f) || frexpf(one, &exponent) != 0.5f || exponent < -20 || exponent > 20) continue;
        bool ok = true;
        for (int i = 0; i < 256 && ok; ++i) {
            double v;
            p.mx_remap[i] = (uint8_t)i;
            if (format_value(format, i, v)) { ok = (double)values[i] == v * one; continue; }
            ok = false;
            for (int j = 0; j < 256 && !ok; ++j)
                if (format_value(format, j, v) && (double)values[i] == v * one) { p.mx_remap[i] = (uint8_t)j; ok = true; }
        }
        if (!ok) continue;
        p.mx_format = format;
        p.mx_factor = one;
        return;
    }
}

namespace {

// A short k under many rows: a workgroup of the matrix form lives for a run or two per wavefront, and the table kernels'
// larger workgroups go through such a matrix faster.  The lines beyond which they do, in rows (times passes over 16 columns
// of X) per compute unit; each lies between shapes measured on its two sides
// (near a line either may be ahead by a tenth or two: the table kernels' forms change in steps).  us, tables / matrix form: one fp16 column,
// 49152 x 128 4.9 / 4.1, 65536 x 128 5.0 / 5.2, 300000 x 128 6.3 / 18; 65536 x 256 8.1 / 6.1, 100000 x 256 6.5 / 8.4; 180000 x
// 640 level, 300000 x 640 25 / 29, 600000 x 1024 level, 1000003 x 1024 78 / 102.  Eight columns: 49152 x 128 6.5 / 5.3, 65536 x
// 128 6.6 / 7.3; 180000 x 640 1.14 : 1, 600000 x 640 71 / 92.  More columns: 49152 x 64 x 33
// 1.5 : 1, 57000 x 64 x 48 10.2 / 23.2 (a run and more of 16-bit and int8 activations goes to the tile kernel, which has a line of its own).
// A k that is no whole number of runs adds loads of single elements and counts for more: 156556 x 754 15.8 / 17.3, int8
// 180000 x 640 1.3 : 1 but 182415 x 692 19.2 / 23.0.
enum { kHalf = 1, kFloat = 2, kBytes = 4, kAny = 7, kRagged = 8 };
// (types of X: fp16 and bf16, fp32, int8; only where k is not a multiple of 128)
struct ShortLine { int k_from, k_to, b_from, b_to, types, rows, to_rows = 1 << 30; };
constexpr int kAllColumns = 1 << 30;
constexpr ShortLine kShort4[] = {
    // k up to a run, two runs
    {1, 128, 1, 1, kAny, 240},            {1, 128, 2, 2, kBytes, 384},          {1, 256, 1, 1, kBytes, 376},
    {1, 256, 1, 2, kHalf | kFloat, 288},  {1, 256, 2, 4, kFloat, 240},          {1, 128, 3, 4, kHalf, 352},
    {1, 128, 5, 8, kHalf, 248},           {1, 64, 5, 8, kFloat, 240},           {1, 128, 9, 16, kHalf, 352},
    {1, 128, 9, 16, kBytes, 400},         {1, 32, 9, 32, kFloat, 100},          {1, 64, 9, kAllColumns, kFloat, 184},
    {65, 128, 9, 16, kFloat, 192, 300},   {65, 128, 17, 32, kFloat, 150},       {1, 64, 17, 32, kBytes, 432},
    {1, 64, 17, kAllColumns, kAny, 600},  {65, 127, 17, kAllColumns, kHalf, 352},
    {65, 128, 17, kAllColumns, kBytes, 352},
    // up to eight
    {513, 768, 1, 1, kHalf | kRagged, 600},  {513, 768, 1, 1, kBytes | kRagged, 416},  {513, 768, 3, 8, kBytes | kRagged, 640},
    {513, 768, 1, 1, kHalf | kFloat, 1024},  {513, 768, 1, 1, kBytes, 3072},    {769, 1024, 1, 1, kHalf | kFloat, 3072},
    {513, 1024, 2, 2, kFloat, 3072},      {513, 640, 2, 4, kHalf, 3400},        {513, 768, 5, 8, kHalf, 900},
    {769, 1024, 5, 8, kHalf, 3072},       {513, 768, 9, 16, kHalf | kBytes | kRagged, 1536},  {513, 640, 9, 16, kHalf | kBytes, 3072},
};
constexpr ShortLine kShort8[] = {  // 8-bit codes
    {1, 64, 1, 1, kAny, 184},    {65, 128, 1, 1, kAny, 288},    {129, 256, 1, 1, kAny, 448},  {257, 512, 1, 1, kAny, 288},
    {513, 768, 1, 1, kAny, 320}, {769, 1024, 1, 1, kAny, 3072}, {769, 1024, 1, 1, kAny | kRagged, 1024},
    {1, 64, 2, 2, kAny, 288},    {1, 32, 5, 16, kFloat, 320},   {1, 32, 17, kAllColumns, kFloat, 320},
    {1, 64, 17, kAllColumns, kAny, 640}, {65, 96, 33, kAllColumns, kAny, 900},
};
bool short_k(const Plan& p, int64_t k)
{
    const int type = p.x_dtype == MSGEMM_F32 ? kFloat : p.x_dtype == MSGEMM_I8 ? kBytes : kHalf;
    const int64_t rows = p.m * ((p.b + 15) / 16);
    const auto beyond = [&](const ShortLine& l) {
        return k >= l.k_from && k <= l.k_to && p.b >= l.b_from && p.b <= l.b_to && (type & l.types) && rows > (int64_t)l.rows * p.cus &&
               rows <= (int64_t)l.to_rows * p.cus &&
               (!(l.types & kRagged) || k % kRun != 0);
    };
    if (p.codes8) return std::any_of(std::begin(kShort8), std::end(kShort8), beyond);
    return std::any_of(std::begin(kShort4), std::end(kShort4), beyond);
}

}  // namespace

// Whether the library's own choice for a plan is the matrix form, and its shape.  anyway: also where the table kernels are the
// faster ones.
bool matrix_choose_shape(Plan& p, int requested_variant, bool anyway)
{
    const msgemm_plan_options_t& o = p.opt;
    p.matrix = false;
    // 8-bit codes: of a format the device converts, and an even number of columns (internally two count for one)
    const bool bytes = p.codes8;
    if (bytes ? p.mx_format == kInt4 || p.k % 4 : requested_variant != MSGEMM_VARIANT_AUTO || p.d != 2) return false;
    const int64_t k = bytes ? p.k / 2 : p.k, code_bytes = p.m * (p.k / 2);
    if ((bytes ? p.scale_group / 2 : p.scale_group) % kRun != 0) return false;
    const bool asked = o.batched_form == 3;
    // a request for a form of the table kernels keeps them
    if (!asked && (o.panels_per_workgroup || o.k_tiles_per_workgroup || o.reduce_mode || o.rows_per_lane || o.no_xcd_map ||
                   o.batched_form == 1 || o.batched_form == 2 || o.batched_segments || o.batched_deal || o.poll_limit || o.skip_publish))
        return false;
    const int64_t runs = (k + kRun - 1) / kRun;
    if (runs * 16384 >= (int64_t)kPastEnd - 65536) return false;  // 32-bit offsets within a row group
    // More than 16 columns (fp32: never, its activations have three parts): the tile kernel, which decodes a code once for 64 columns,
    // where its row groups and column tiles fill five eighths of the device; passes of the streaming kernel over 16 columns at a time
    // where they do not, until the codes of all passes are many.  us, passes / tile.  Filling: 16384 x 128 x 20 fp16 3.9 / 3.9, x 64 5.8 / 4.6;
    // 11008 x 512 x 20 4.7 / 4.5, x 64 7.1 / 5.5; 14336 x 4096 x 17 13.7 / 12.6; 8192 x 4096 x 72 24.7 / 15.0; 28672 x 4096 x 64 45.9 / 22.1.  Not: 4096 x 4096 x
    // 64 (32 MiB) 8.0 / 13.7, 8192 x 4096 x 64 (64) 13.2 / 14.2, 4096 x 14336 x 48 (84) 19.1 / 18.0, 8192 x 8192 x 48 (96) 26.2 / 19.0; int8 4096 x 14336 x 64
    // (112) 14.6 / 14.7, 8192 x 7168 x 64 (112) 16.0 / 14.8, 8192 x 8192 x 64 (128) 17.5 / 15.9; 8-bit codes 8192 x 4096 x 20 fp16 (64) 13.4 / 13.9, 8192 x 4096 x 48 (96) 19.7 / 16.2.
    // int8 up to 48 columns: a long k keeps the kernel of smaller tiles (28672 x 4096 x 24 14.6 / 15.6, 14000 x 3006 x 33 10.8 / 11.7; 20 runs and more were
    // compared) by its own lines; a short one under few rows does well with passes (16384 x 512 x 20 4.2 / 4.3, 16384 x 1024 x 20 5.3 / 5.1).
    const bool tile_can = p.b > 16 && p.x_dtype != MSGEMM_F32 && k >= kRun &&
                          !(p.x_dtype == MSGEMM_I8 && k > ((int64_t)1 << 17));  // (int8 sums are 16 x too large in 32 bits)
    const bool int8 = p.x_dtype == MSGEMM_I8, narrow8 = int8 && p.b <= 48;
    const int64_t pass_mib = ((p.b + 15) / 16 * code_bytes) >> 20, row_groups = (p.m + 63) / 64;
    const int small_tiles = p.b <= 32 ? 2 : 3;
    const bool small = tile_can && narrow8 && (asked && o.rows_per_lane ? o.rows_per_lane == 4 :
        runs >= 20 && pass_mib >= (row_groups * 8 > (int64_t)5 * p.cus && p.b >= 10 * small_tiles ? 48 : 112));
    // (tiles of 32 columns or of 64, whatever is padding.  us, against tiles of 48 columns and 16 rows where those fitted better: 28672 x 8192 x 40 fp16 41.8 / 45.0, bf16 with
    // scales 45.2 / 53.0, 14336 x 4096 x 33 14.8 / 18.0; 65 to 96 columns, two passes of 64 against two of 48: 28672 x 8192 x 80 69.7 / 92.2, 11008 x 2048 x 72 12.4 / 19.6,
    // int8 28672 x 8192 x 72 50.2 / 58.0)
    const int64_t tall_passes = p.b <= 32 ? 1 : (p.b + 63) / 64;
    const bool tall = tile_can && !small && (asked && o.rows_per_lane ? o.rows_per_lane == 4 :
        row_groups * tall_passes * 8 > (int64_t)5 * p.cus ? !narrow8 || runs >= 8 || row_groups > 2 * p.cus : !narrow8 && pass_mib >= (int8 ? 112 : 80));
    const bool tile = small || tall;
    const int tile_tiles = small ? small_tiles : p.b <= 32 ? 2 : 4;
    const int64_t tile_passes = (p.b + 16 * tile_tiles - 1) / (16 * tile_tiles);
    // One fp32 column of 4-bit codes: decoding and three products per weight where the table kernels add once per pair
    // (4096 x 4096 5.5 us against 6.9, 8192 x 8192 11.0 against 10.3, 49152 x 12288 74 against 52; 8-bit codes, one
    // conversion for two, 12.5 against 17.0 at 8192 x 8192).
    if (p.x_dtype == MSGEMM_F32 && p.b == 1 && !bytes && p.m * k > ((int64_t)32 << 20) && !asked && !anyway) return false;
    // (streaming kernel, 300001 x 512: 19 us against 27, 300001 x 64: 6.3 against 17; ahead at 100000 rows and 512 columns,
    // 17.2 against 20.5 with eight columns of X)
    if (!tile && k <= 512 && p.m > (int64_t)512 * p.cus && !asked && !anyway) return false;
    // (tile kernel: short k is no matter to it until there are very many workgroups of one run; us, tables / tile: 49152 x 128 x 20 fp16 17.0 /
    // 5.0, 80000 x 256 x 64 31.4 / 13.5, 300000 x 128 x 64 60 / 42, bf16 with scales 67 / 55; 1000000 x 128 x 17 61 / 81, x 33 105 / 115)
    if ((tall ? runs == 1 && p.m > (int64_t)2400 * p.cus : short_k(p, k)) && !asked && !anyway) return false;

    const bool compact = p.b <= (p.x_dtype == MSGEMM_I8 ? 8 : 4);
    const bool scaled = p.scale_group > 0;
    const int Wr = tile ? 4 : 1;   // (wavefronts of 16 R rows, or half as many of 32 R)
    const int width = tile ? 3 : compact ? 0 : p.b <= 8 ? 1 : 2;
    p.mx_cols = tile ? tile_tiles : 2 * width;
    const int64_t passes = tile ? tile_passes : (p.b + 15) / 16;
    if (passes > 65535) return false;
    const auto groups = [&](int r) { return (p.m + 16 * Wr * r - 1) / (16 * Wr * r); };
    // (wavefronts that the rule for segments counts with; the streaming kernel's workgroups may have more)
    const auto waves = [&](int r) { return tile ? 8 : width == 2 && r == 4 ? 8 : 4; };
    // Few row groups and a long k: segments of it side by side, their sums added by a second launch, as long as a wavefront
    // keeps 16 runs (tile kernel: a workgroup 20.  Uncut / two segments / four: 4096 x 14336 x 64 fp16 37.5 / 25.0 / 18.5 us, 8192 x 8192 x 64 24.3 / 19.9, bf16 with scales
    // 26.4 / 20.3, 6144 x 6144 x 64 (24 runs each) 19.2 / 15.2, 8192 x 5120 x 64 (20) 16.7 / 15.3, 8192 x 4096 x 64 (16) 14.3 / 14.1, x 32 11.6 / 11.0; where there are
    // more than half as many row groups as compute units 11008 x 4096 x 64 14.7 / 21.9).  With fp32 activations a
    // run takes three products and as much splitting, and fewer are enough: 448 x 12288 x 1 9.6 us uncut, 8.0 in two, 7.2 in four
    // segments of 6 runs a wavefront, 448 x 4096 x 1 4.9 uncut, 6.1 in two; 448 x 8192 x 16 16.0, 12.0 and 9.4, 448 x 4096 x 16 9.6,
    // 8.7 and 7.5, x 8 6.8, 7.1 and 6.6.
    const int keep = tile ? 20 : p.x_dtype != MSGEMM_F32 ? 16 : compact ? 6 : p.b <= 8 ? 5 : 4;
    const auto segments_of = [&](int r) {
        int64_t n = 1;
        while (groups(r) * passes * n * 2 <= p.cus && runs >= 2 * n * (tile ? keep : waves(r) * keep)) n *= 2;
        return n;
    };
    // Row tiles per wavefront: the work of the busiest compute unit, in row tiles for the streaming kernel, weighted by
    // what a row tile costs -- the fewer tiles share a load of activations, the more of it each carries (measured with
    // 1, 4 / 8 and 16 columns) -- and in workgroups of 1, 2 and 3 tiles for the tile kernel (a round of one tile 15.2 us, of two 22, of three 32: 16384 x 4096 x 64 fp16 in one
    // round of one tile 16.2, 28672 x 4096 x 64 in one, two and three tiles 29.5, 23.6 and 27.9, 40960 x 4096 x 64 45.3, 41.8 and 31.9, 49152 x 12288 x 64 127, 114 and 82, 28672 x 8192 x 64 bf16
    // with scales 58.9 and 45.1; three scaled tiles do not fit the registers).
    const int tiles[2][3] = {{1, 2, 4}, {1, 2, 3}};
    double cost[4][3] = {{1.25, 2.0, 4.12}, {1.2, 2.0, 3.8}, {1.55, 2.4, 4.0}, {1.0, 1.35, 1.9}};
    // (a column or a few of 16 bits are a small load: one row tile costs its share of two where the stream is short, or is one column under four workgroups a
    // compute unit, and more the longer it is and the more columns it has.  us, one tile / two; where two workgroups of one tile do the work of one of two:
    // 16384 x 3840 x 1 fp16 9.4 / 9.6, 7043 x 2176 x 3 with scales (two, or one of two) 4.2 / 4.0, 8192 x 8192 x 1 bf16 8.4 / 8.7, 24089 x 5888 x 1 with scales 14.7 / 14.0, 13160 x 8192 x 2 with scales 13.2 / 12.6, 24089 x 4860 x 4 bf16
    // 15.0 / 13.8, 24089 x 2944 x 4 fp16 with scales 9.9 / 8.8, 40720 x 1280 x 4 7.8 / 7.2, 23552 x 1280 x 3 5.7 / 5.3, 40720 x 2048 x 1 10.2 / 9.5, but 12759 x 896 x 4 bf16 (3.1 tiles of one a compute unit) 3.6 / 3.9, 16384 x 8192 x 4 bf16 with scales 16.2 / 14.3; where they do not: 20480 x 8192 x 1 15.7 / 16.9, 11008 x 4096 x 4 bf16 7.1 / 8.0, 33280 x 8192 x 4 bf16
    // 1.06 : 1.  Over 210 problems with 6056 to 33280 rows and 1, 2 and 4 columns the choice takes 0.6 percent more than the faster of
    // the two in the mean, 9 at most.
    // fp32, two tiles / four: 16384 x 8192 x 4 19.2 / 18.6, 33280 x 4096 x 16 38.0 / 34.3)
    if (width == 0 && !bytes && p.x_dtype != MSGEMM_F32 && !int8)
        cost[0][0] = groups(1) <= 2 * p.cus && runs < 64 ? 1.05 : scaled && runs < 24 && groups(1) > 4 * p.cus ? 1.10 : runs < 24 || (p.b == 1 && runs < 72 && groups(1) <= 4 * p.cus) ? 0.98 : runs >= (p.b > 2 ? 48 : 96) ? 1.25 : 1.05;
    if (p.x_dtype == MSGEMM_F32 && !bytes) cost[0][2] = 3.95, cost[2][2] = 3.8;
    double best = 0;
    int R = 1;
    const int sizes = tile && bytes && scaled && tile_tiles > 2 ? 1 : (tile && scaled) || bytes ? 2 : 3;   // (what the registers hold)
    for (int i = 0; i < sizes; ++i) {
        const int r = tiles[tile][i];
        const int64_t n = tile ? segments_of(r) : 1;
        const double c = (double)((groups(r) * passes * n + p.cus - 1) / p.cus) * cost[width][i] / (double)n;
        if (i == 0 || c < best) { best = c; R = r; }
    }
    for (int i = 0; i < sizes; ++i)
        if (asked && o.panels_per_workgroup == tiles[tile][i]) R = o.panels_per_workgroup;
    int64_t segments = segments_of(R);
    // (a single fp32 column whose chains stay long although they are cut: 2048 x 16084 10.2 us in two segments, tables 8.7;
    // level at 2048 x 12288, 12 runs a wavefront)
    if (p.x_dtype == MSGEMM_F32 && p.b == 1 && !bytes && segments > 1 && runs > segments * waves(R) * 12 && !asked && !anyway) return false;
    if (asked && o.batched_segments) segments = o.batched_segments < runs ? o.batched_segments : runs;
    // Streaming kernel, wavefronts and depth of their rings.  A compute unit's share of 6.3 TB/s over a trip of a microsecond is 24 KiB of codes; the forms
    // chosen have 16 (a short k: an unrolled loop that is gone through once or twice is fetched for nothing) to 64 KiB in flight, 32 where there is one
    // workgroup of one row tile and a long k.  us, "wavefronts x depth", one column or a few and one row tile:
    //   a workgroup per compute unit, 4 x 8 / 8 x 4 / 16 x 2 (a wavefront short of a whole ring asks for less, so which is ahead changes with the
    //   length: the lines follow 21 lengths of 32 to 158 runs and more beyond).  fp16 7.61 / 7.28 / 7.41 at 4096 x 14336 x 1, 8.74 / 8.48 / 8.67 at 18432; 4096 x 7168 x 1 5.22 / 4.92 /
    //   4.94, 3072 x 7168 x 2 4.86 / 4.58 / 4.50; rings that come out even, 4096 x 8192 x 1 5.20 / 5.23 / 5.40, 3072 x 12288 x 2 6.07 / 6.13 / 6.22; 4096 x 24576 x 4 11.9 / 12.1 / 12.3.  fp16 with
    //   scales: 4096 x 4096 x 1 4.11 / 3.98 / 3.82, 4096 x 14336 x 2 7.33 / 7.17 / 7.21, 4096 x 14336 x 1 7.92 / 7.52 / 7.65, x 4 8.45 / 8.52 / 8.58, 4096 x 18432 x 4 10.0 / 10.2 / 10.5, 3072 x 40960 x 2
    //   16.6 / 16.2 / 16.3.  bf16 with scales: 3072 x 11264 x 2 6.79 / 6.38 / 6.05, 4096 x 40960 x 1 18.5 / 17.9 / 18.0.  int8, columns of whole 16-byte pieces: 4096 x 3328 x 1 3.54 / 3.39 / 3.58, 4096 x
    //   5904 x 1 5.33 / 5.29 / 5.09, 4096 x
    //   7168 x 1 4.80 / 4.72 / 4.86, 3864 x 14336 x 3 7.21 / 6.79 / 6.64; others: 3072 x 7382 x 2 6.62 / 6.78 / 7.43, 3864 x 11940 x 3 7.43 / 7.82 / 7.75, 4096 x 11942 x 4 9.2 / 9.6 / 10.8, 3072 x 4996 x 2 4.11 / 4.12 / 4.02.  Five to eight int8 columns: 4 x 8 / 4 x 4 4096 x
    //   4096 x 8 4.3 / 3.9, 2560 x 14336 x 8 level.  fp32 4 x 8 / 4 x 4 / 16 x 2: 4096 x 4096 x 1 5.3 / 4.7 / 4.6, 3072 x 40960 x 4 27.0 / 25.5 / 22.8.
    //   A short k, 4 x 8 / 4 x 4 / 4 x 2: 3072 x 1024 x 1 fp16 3.0 / 2.7 / 2.5, int8 2.8 / 2.6 / 2.5, 3072 x 1290 x 1 fp16 3.1 / 2.9 / 3.1, int8 3.6 / 3.3 / 3.7, 3072 x 2048 x 1 fp16
    //   3.3 / 2.9 / 3.2; int8 3072 x 2816 x 1 3.15 / 3.25 / 3.6, x 8 3.5 / 3.4 / 3.7, 3072 x 2580 x 1 3.9 / 4.3 / 5.0, 3072 x 3070 x 1 4.0 / 4.4 / 5.1, 3072 x 2820 x 4 3.6 / 3.8 / 4.2, 3072 x 3334 x
    //   1 3.8 / 4.0, 3072 x 3596 x 2 4.2 / 4.6, 3072 x 3686 x 3 4.4 / 4.7, but 3072 x 2178 x 1 3.2 / 3.1 / 3.5, 3072 x 3334 x 4 (k no multiple of four) 4.3 / 4.2
    //   two: 8192 x 8192 x 1 bf16 4 x 8 9.1, 4 x 4 8.4; 8192 x 14336 x 1 fp16 11.8, 11.4
    //   three and more: 11003 x 4098 x 1 fp16 4 x 8 7.5, 4 x 2 6.9; 11008 x 4096 x 4 bf16 8.4, 7.1; 20000 x 8192 x 4 int8 4 x 4 15.7, 4 x 2 16.9; 12093 x
    //   20842 x 1 int8 4 x 8 22.6, 4 x 4 23.3; 12288 x 4096 x 1 int8 4 x 4 6.5, 4 x 2 6.0, with columns that end inside a 16-byte piece 12288 x 3640 x 1 6.7, 7.1, 9000 x 5900 x 2 8.0, 8.3
    // Two row tiles: 6144 x 6144 x 3 fp16 4 x 4 5.6; in more workgroups 42240 x 6912 x 4 fp16 4 x 4 27.9, 8 x 2 27.5, 13160 x 24704 x 1 bf16 31.7, 30.8, 33792 x
    // 1792 x 1 fp16 4 x 4 8.5, 8 x 2 8.4, 4 x 2 8.1, 33280 x 7424 x 3 fp32 4 x 4 35.9, 8 x 2 35.4, 4 x 2 35.0; with scales, three runs a wavefront, 46335
    // x 1408 x 1 fp16 4 x 4 7.9, 4 x 2 8.3, bf16 8.9, 8.9, but 46335 x 1024 x 1 7.3, 7.0, 24089 x 1792 x 1 6.5, 6.3.  int8, 4 x 4 / 8 x 2 / 4 x 2: 37725 x
    // 3640 x 1 14.3 / 19.0 / 16.3, 19847 x 6744 x 1 14.4 / 17.9 / 14.2, 37725 x 6744 x 4 23.9 / 26.9 / 26.2, 32760 x 9900 x 1 (78 runs) 27.1 / 28.4, 26000 x 10240 x 4 25.2 / 24.6 / 26.1, 26000 x 20842 x 8 62.2 /
    // 60.9 / 61.5; a k that is no whole number of runs 22868 x 18240 x 4 36.3 / 38.2; two workgroups, 14848 x 10240 x 1 13.7 / 14.3 / 13.7, 14848 x 40192 x 1 48.0 / 50.4 / 48.1.
    // Wider operands: 8192 x 8192 x 16 int8 4 x 4 8.8, 8 x 2 8.3; 28672 x 4096 x 6 fp16 (four row tiles) 4 x 3 14.4, 8 x 2 13.2; four row tiles and 16
    // columns, whose operands fill the LDS ports, 14336 x 4096 x 16 8 x 2 9.5, 4 x 2 9.0, 11264 x 4096 x 16 9.1, 8.7, 8960 x 4096 x 16 (140 workgroups) 8.8, 8.5, 11264 x 8192 x 16
    // 14.8, 14.6, 9216 x 8192 x 16 level, but 4107 x 908 x 32 5.0, 5.3, and 8679 x 8064 x 16 bf16, for half the compute units, 14.5, 15.5; int8 10240 x 4096 x 16 7.2, 7.3, 13312 x
    // 4096 x 16 7.6, 7.7, level at 14336, 26000 x 3072 x 16 12.3, 11.1, in passes 8192 x 8192 x 24 11.6, 10.3, but where k is no
    // whole number of runs 7970 x 2720 x 32 8.3, 9.0, 16000 x 2720 x 16 8.4, 9.2, 8192 x 3000 x 20 7.35, 8.2 (two workgroups a compute unit, 26000 x 3000 x 16 15.1, 13.6); 16 bits in passes 8192 x 4096 x 32 8.7, 8.3, 4096 x 4096 x 64 8.3, 8.2, but three and more over a long k 4096 x 5376 x 64 9.5, 9.8, 5120 x 8192 x 40
    // 12.4, 12.7, two with bf16 and scales 5120 x 14336 x 24 20.0, 22.1, 6144 x 5120 x 24 10.0, 10.2 (but 8192 x 4096 x 32 9.3, 9.0), or fewer columns with scales over a long k 11776 x 17152 x 11 fp16 27.2,
    // 28.5, bf16 28.3, 29.9, 11008 x 9216 x 9 16.2, 17.4, 9472 x 7680 x 11
    // 14.8, 15.1, x 13 level, 15907 x 4608 x 11 level; fp16 in two passes of two row tiles 4 x 4 / 8 x 2: 4096 x 14336 x 20 14.2 / 14.9, 3584 x 18944 x 22 17.7 / 18.7, x 24 with scales 17.4 / 18.0, but 4096 x 6144 x 22 7.8 / 7.3, bf16
    // with scales 4096 x 14336 x 22 16.3 / 14.6; int8 in two row tiles over a short k 4 x 2 / 8 x 2: 9984 x
    // 1536 x 24 5.5 / 6.5, 18176 x 1536 x 16 6.0 / 6.4, but 18176 x 3072 x 16 9.4 / 8.9; int8 over a long k
    // that is no whole number of runs (columns of X then start anywhere in a line of the caches) 4 x 4 / 8 x 2: 4000 x 11428 x 16 11.8 / 12.5, 5608 x 11426 x 9 13.7 / 14.3, 2000 x 17326 x 32 16.3 / 17.0, but 4000 x
    // 5620 x 16 7.6 / 7.2, 5608 x 17408 x 16 16.7 / 16.5; 14336 x 4096 x 8 in
    // two row tiles, two workgroups a compute unit, 9.0, 8.55; fp32, whose operands of eight
    // wavefronts take 96 KiB of LDS, 4096 x 4096 x 8 4 x 2 7.2, 8 x 2 6.4, 38400 x 3840 x 6 29.9, 36.5.
    const int64_t per_cu = (groups(R) * passes * segments + p.cus - 1) / p.cus, seg_runs = runs / segments;
    const bool f32 = p.x_dtype == MSGEMM_F32;
    // (int8, one or three columns, or up to four at addresses that are multiples of four: others are bound by the loads of the activations themselves)
    const bool few8 = int8 && p.b <= 4 && (p.b % 2 == 1 || k % 4 == 0);
    int W = 4, D = 2;
    if (tile) {
        W = 8;
    } else if (bytes) {
        D = compact ? 4 : width == 1 && R == 1 && !f32 ? 4 : 2;
    } else if (!compact) {
        const bool bf16_scales = scaled && p.x_dtype == MSGEMM_BF16, part = scaled && p.b % 16 != 0 && p.b % 16 < 12;
        const int64_t end = passes > 2 || (passes == 2 && bf16_scales) ? 40 : part ? (passes == 1 ? 60 : 100) : runs + 1;
        const bool full = groups(R) * passes * 16 >= (int8 ? 14 : 9) * p.cus && seg_runs < end && !(int8 && k % kRun != 0 && per_cu == 1);
        W = f32 ? (per_cu == 1 && seg_runs >= 16 ? 8 : 4) : (width == 2 ? R == 4 && seg_runs >= 16 && full : R == 2 && per_cu > 1) ? 4 : 8;
        if (p.x_dtype == MSGEMM_F16 && width == 2 && R == 2 && passes == 2 && per_cu == 1 && seg_runs >= 80) W = 4, D = 4;
        if (int8 && R == 2 && per_cu > 1 && seg_runs < 16) W = 4;
        if (int8 && width == 2 && R < 4 && k % kRun != 0 && seg_runs >= 80) W = 4, D = 4;
    } else if (R == 2) {
        if (per_cu == 1 || (int8 && (per_cu == 2 || seg_runs < 80 || k % kRun != 0)) || (scaled && !f32 && seg_runs > 8 && seg_runs <= 12)) D = 4;
        else if (!f32 && seg_runs >= 28) W = 8;
    } else if (R == 1) {
        const bool bf16 = p.x_dtype == MSGEMM_BF16, pieces = k % 16 == 0;
        const int64_t end = f32 || (scaled && p.b <= 2) ? runs + 1 : 160;
        if (per_cu == 1 && int8 && p.b <= 4 && seg_runs >= (pieces ? 26 : 32) && seg_runs < end) {
            if (seg_runs > 32 && seg_runs < 50) W = 16;
            else if (pieces) W = 8, D = 4;
            else D = 8;
        } else if (per_cu == 1 && !int8 && seg_runs >= 32 && seg_runs < end) {
            const bool wide = bf16 && scaled ? p.b > 1 || seg_runs < 160 : seg_runs < 92 && (scaled || seg_runs % 32 != 0);
            if (f32 || wide) W = 16;
            else if (scaled && p.b > 2 && seg_runs >= 108) D = 8;
            else W = 8, D = 4;
        } else if (seg_runs >= (int8 ? 80 : 128) && !f32) D = 8;
        else if (per_cu == 1 && seg_runs >= 20 && seg_runs < 32 && few8) D = 8;
        else if (seg_runs >= (per_cu > 2 ? (few8 && k % 16 != 0 ? 28 : 48) : f32 ? 16 : 11)) D = 4;
    }
    p.mx_depth = D;
    p.mx_tile_kernel = tile;
    p.mx_r = R;
    // (int8, more than 48 columns: from 66 runs a segment the kernel of smaller tiles is ahead, whose wavefronts along k are fewer; in passes only where the
    // workgroups leave compute units idle in their last round.  us, smaller / larger: 27648 x 10752 x 50 36.2 / 40.7, x 64 38.8 / 40.4, 36864 x 9216 x 50 40.2 / 42.9, 49152 x 12288 x 64
    // 60.8 / 62.6, 16384 x 20480 x 50 (two segments of 80) 42.4 / 44.1; 27648 x 8192 x 50 32.5 / 31.4, x 4096 19.3 / 17.9, 12288 x 20480 x 64 (four of 40) 38.7 / 36.8; two passes, 36864 x
    // 10752 x 80 (384 workgroups) 74.1 / 79.9, 27648 x 10752 x 100 59.8 / 63.2, three, 28672 x 9216 x 150 (450) 66.5 / 69.8, 16384 x 14336 x 80 (256) 45.5 / 44.6, 49152 x 10752 x 80 (512) 93.8 / 90.8)
    p.mx_tall = tall && !(int8 && p.b > 48 && seg_runs >= 66 && (passes == 1 || groups(R) * passes * segments * 16 <= 15 * p.cus * per_cu));
    p.mx_row_waves = p.mx_tall ? kTileRowWaves : Wr;
    p.mx_waves = W;
    p.mx_segments = (int)segments;
    p.matrix = true;
    p.row_blocks = groups(R);
    p.m_pad = p.row_blocks * 16 * Wr * R;
    p.ktiles = runs;
    p.fs.groups = bytes ? kRun : kRun / 2;
    p.fs.cols = 1;
    p.fs.entry_bytes = 4;
    p.fs.tile_rows = 16 * Wr * R;
    const int64_t sums = (int64_t)(W / p.mx_row_waves) * segments;
    p.segments = (int)(runs < sums ? runs : sums);  // partial sums per output: one per wavefront (or group) with a run
    p.partial_bytes = segments > 1 ? (size_t)segments * (size_t)p.b * (size_t)p.m_pad * 4u : 0;
    return true;
}

static int scale_slots(const Plan& p) { return p.mx_r == 3 ? 4 : p.mx_r; }
size_t matrix_scale_bytes(const Plan& p)
{
    return (size_t)p.nblocks * (size_t)p.row_blocks * (size_t)(p.mx_row_waves * (p.mx_tall ? 32 : 16) * scale_slots(p)) * 2u;
}

static int matrix_repack(const Plan& p, uint8_t* row_major, bool inverse, hipStream_t s)
{
    const int64_t dwords = p.ktiles * p.m_pad * 16;
    int64_t blocks = (dwords + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    const auto kernel = inverse ? (p.mx_tall ? matrix_repack_kernel<true, true> : matrix_repack_kernel<true, false>)
                                : (p.mx_tall ? matrix_repack_kernel<false, true> : matrix_repack_kernel<false, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(256), 0, s, row_major, p.codes_tiled, p.m, p.k, p.ktiles,
                       p.mx_r * p.mx_row_waves, encoding_of(p.x_dtype), dwords);
    MSGEMM_HIP_TRY(hipGetLastError());
    return MSGEMM_OK;
}

size_t matrix_code_bytes(const Plan& p) { return (size_t)p.ktiles * (size_t)p.m_pad * (p.codes8 ? 128u : 64u); }

int matrix_repack(const Plan& p, const void* W_codes, hipStream_t s)
{
    if (p.scales) {
        const int64_t total = (int64_t)(matrix_scale_bytes(p) / 2);
        int64_t blocks = (total + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(p.mx_tall ? matrix_repack_scales_kernel<32> : matrix_repack_scales_kernel<16>, dim3((unsigned)blocks), dim3(256), 0, s,
                           (const __half*)p.scales, (__half*)p.scales_ordered, p.m, p.nblocks, p.mx_r, p.mx_row_waves, scale_slots(p), total);
        MSGEMM_HIP_TRY(hipGetLastError());
    }
    if (p.codes8) {
        const int64_t dwords = (int64_t)(matrix_code_bytes(p) / 4);
        int64_t blocks = (dwords + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        Remap remap;
        for (int i = 0; i < 256; ++i) remap.to[i] = p.mx_remap[i];
        hipLaunchKernelGGL(p.mx_tall ? matrix_repack8_kernel<true> : matrix_repack8_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, s,
                           (const uint8_t*)W_codes, p.codes_tiled, p.m, p.k / 2, p.ktiles, p.mx_r * p.mx_row_waves, remap, dwords);
        MSGEMM_HIP_TRY(hipGetLastError());
        return MSGEMM_OK;
    }
    return matrix_repack(p, (uint8_t*)W_codes, false, s);  // (read only in this direction)
}

int matrix_unpack(const Plan& p, uint8_t* row_major, hipStream_t s) { return matrix_repack(p, row_major, true, s); }

int launch_matrix(const Plan& p, const void* X, int64_t ldx, void* Y, int64_t ldy, hipStream_t s)
{
    MatrixArgs a;
    a.codes = p.codes_tiled;
    a.scales = (const __half*)p.scales_ordered;
    a.X = X; a.ldx = ldx; a.Y = Y; a.ldy = ldy;
    const int64_t k = p.codes8 ? p.k / 2 : p.k, group = p.codes8 ? p.scale_group / 2 : p.scale_group;
    a.m = p.m; a.k = k; a.b = (int)p.b;
    a.runs = (int)p.ktiles;
    a.full_runs = (int)(k / kRun);
    a.nblocks = (int)p.nblocks;
    a.partials = p.mx_segments > 1 ? (uint32_t*)p.partials : nullptr;
    a.m_pad = p.m_pad;
    a.seg_runs = ((p.mx_tile_kernel ? a.runs : a.full_runs) + p.mx_segments - 1) / p.mx_segments;
    a.row_groups = (int)p.row_blocks;
    a.passes = p.mx_tile_kernel ? (int)((p.b + 16 * p.mx_cols - 1) / (16 * p.mx_cols)) : (int)((p.b + 15) / 16);
    a.div_block = make_fastdiv(group > 0 ? (uint32_t)(group / kRun) : 1u);
    a.factor = p.codes8 ? (p.x_dtype == MSGEMM_F16 ? p.mx_factor : 1.0f) : p.x_dtype == MSGEMM_BF16 ? 16.0f : 1.0f;
    a.times = p.codes8 ? p.mx_factor : 1.0f;
    if (p.codes8) {
        switch (p.x_dtype) {
        case MSGEMM_F16: return launch_for_format<__half>(p, a, s);
        case MSGEMM_BF16: return launch_for_format<bf16_t>(p, a, s);
        case MSGEMM_F32: return launch_for_format<float>(p, a, s);
        default: return MSGEMM_ERR_UNSUPPORTED;
        }
    }
    if (p.mx_tall) {
        switch (p.x_dtype) {
        case MSGEMM_F16: return launch_tile_for_type<__half>(p, a, s);
        case MSGEMM_BF16: return launch_tile_for_type<bf16_t>(p, a, s);
        case MSGEMM_I8: return launch_tile_for_type<int8_t>(p, a, s);
        default: return MSGEMM_ERR_UNSUPPORTED;
        }
    }
    if (p.mx_tile_kernel) return p.x_dtype == MSGEMM_I8 ? launch_small_tile(p, a, s) : MSGEMM_ERR_UNSUPPORTED;
    switch (p.x_dtype) {
    case MSGEMM_F16: return launch_for_type<__half>(p, a, s);
    case MSGEMM_BF16: return launch_for_type<bf16_t>(p, a, s);
    case MSGEMM_F32: return launch_for_type<float>(p, a, s);
    case MSGEMM_I8: return launch_for_type<int8_t>(p, a, s);
    default: return MSGEMM_ERR_UNSUPPORTED;
    }
}

}  // namespace msgemm

// Dense tiles on 32x32x16 MFMAs (gfx950): every (query, key) pair of a head visited
// once, out = sum over the pairs of a weight times a row.
//
//   YOSO-E forward     Y  = P V                         P = (1 - arccos(cos)/pi)^tau
//   YOSO-E backward    dV = P^T dY,  dQ = (tau/2) [(dY V^T) .* P] K,  dK likewise
//   YOSO backward      dV = (1/m) C^T dY, dQ = tau/(2m) [(dY V^T) .* C] K, dK likewise
//   *YOSO backward     dQ = (1/m) [(dY V^T) .* N ./ (pi sqrt(max(1 - x^2, 1/64)))] K, dK
// with C = sum_h B_h (Sec. 3.1, 3.3: the hashes summed first; an integer, at most m)
// and N = sum_h C_h of the sampled true gradient (tau [codes equal] + [one bit apart]).
//
// One workgroup of WAVES waves owns 32 WAVES "fixed" rows of one side, 32 per wave, and
// streams the other side through LDS in tiles of T = 8 WAVES rows.  Per 32 x 32 block of
// (streamed, fixed) pairs: the scalar products on MFMA (x for cosines, G = g . a), the
// weights W on the VALU, and out^T += rows^T W on MFMA again.  The 32 x 32 shape runs at
// 1.8x the rate of the 16 x 16 ones (2.33 against 1.3 PFLOP/s), and a wave's 32 fixed
// rows halve the operand reads of 16.  A block's result layout is the next product's
// operand layout up to the order of the contraction index (below), so weights never
// cross lanes.
//
// What bounds it: the vector units first (13 to 25 vector instructions per pair, of which
// most take 4.4 clocks of a SIMD and only all-register fp32 and three-input bit operations
// 2.5), then the MFMAs (12 to 32 of 32 clocks per 1024 pairs); two waves share a SIMD.  The
// next tile's work (convert and stage its rows, count its pairs) is cut into slices between
// the MFMAs of the present one, so that a wave has both kinds to issue at any time.  Tiles
// and counts are double buffered in LDS: one barrier per tile.
//
// Precision: fp32 operands as fp16 (hi, lo) pairs and three products, as everywhere in
// this library; bf16 operands, scaled by powers of two, are exact as hi alone (cosine rows,
// which are normalised, keep both).  Scales, all powers of two but the first:
//   cosine rows     unit length times 2^4
//   fixed rows a    each row by 2^(6 - e), ||a|| < 2^e (counts: 2^(9 - e) and less)
//   streamed rows   each head's tensor by 2^(13 - e), max |x| < 2^e (found by a first scan); a
//                   tile of 32 or 64 rows far below its head by its own e (YOSO-E; counts up
//                   to kFineRows rows); those that counts alone weight (dV's dY, the
//                   forward's V) dim by dim, as the bucket tables do, with the dims' powers
//                   taken back from a
//   weights         counts: |G| < 2^25 times C 2^-11, a row that meets a count of 4 or more scaled
//                   down (widen); *YOSO: |G| < 2^22, each row to what comes (row_scale);
//                   P by pbase^tau, just below 2^16 (expect_scale), G P by 2^-7 more
#include <type_traits>

#include "common.h"
#include "launch.h"
#include "timing.h"

namespace yoso {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

enum : int { kWeightCount = 0, kWeightStar = 1, kWeightExpect = 2 };
// which sums: the P (or C) weighted one, the G weighted one, or both
enum : int { kSumP = 0, kSumPG = 1, kSumG = 2 };

constexpr float kCosScale = 16.0f;   // cosine rows: unit length times 2^4
constexpr int kFixedExp = 6;         // fixed rows: norm below 2^6
constexpr int kFixedExpCount = 9;    // (weighted by counts: below 2^9, scaled down to 2^4 at most)
constexpr int kCountExp = 11;        // counts: C 2^-11, exact fp16 numbers
constexpr float kNearFloor = 1.0f / 64.0f;  // *YOSO: 1 - x^2 is raised to at least 1/64
// *YOSO: G (|G| < 2^22) enters the weights times 2^-kRowExp, which leaves the product of one
// hash below 2^16.  Many hashes and small angles make a pair's weight up to 650 times that:
// the weights are scaled per row to what comes (row_scale).  (With a scale for the worst that could
// come an ordinary weight lay at 2^-3, 22 bits above the pair's end: dK of keys whose
// queries have dY 10^4 below the head's largest was 7e-4 off, now 2e-5.)
constexpr int kRowExp = 8;
constexpr float kWeightMax = 32768.0f;

// Counts: streamed rows up to which tiles have scales of their own beside their head's, as the
// 16 x 16 form of these lengths has them.  (Where dY of half the rows lies 10^7 below the other
// half's, m = 2, tau = 8, 900 rows: one row of dK in a hundred was 1.3e-3 or more off, now 7e-7.
// The scan with a maximum per tile costs the backward of 384 x 512 1.8%, 1 x 512
// 3%, 192 x 1000 forward 1 to 2%; longer sides nothing beyond 1%.)
constexpr int kFineRows = 1024, kTileRows = 32, kFineTiles = kFineRows / kTileRows;

// Counts, fp32: streamed rows after which the running sums go to the output (or partial output), to
// start again from zero.  A sum over 4096 rows is 128 additions to a running one, and where the
// addends have one sign (clustered rows) their rounding, sqrt(128 / 3) times 0.29 of the last
// place, is most of the error: dQ of 32 x 4096 clustered 2.71e-7, in parts of 2048 rows 2.30e-7 (the
// pair passes 2.49e-7); m = 64 2.76e-7, in parts of 1024 2.15e-7 (2.32e-7).  Backward of 32 x 4096 1.06 ->
// 1.09 ms, m = 48, whose registers spill more with it, 1.61 -> 1.76.  (dK and dV of twelve plane words
// spill 50 more and are no less precise than the pairs: 2.60e-7 and 2.65e-7.)
template <int NW>
constexpr int kFlushRows = NW == 16 ? 1024 : 2048;

struct TileSide {
    const void *fx, *fa;         // fixed side: cosine (or x) rows, rows of G
    const void *sx, *sg, *sy;    // streamed side: cosine rows, rows of G, rows summed
    const uint32_t *fpl, *spl;   // bit planes of the codes [bh][n][NW] (C, N; backward)
    const uint16_t *fcodes, *scodes;  // the codes [bh][n][m] themselves (forward, which has no scratch for planes)
    void *out_p, *out_g;         // P- (C-) weighted sum of sg (forward: of sy); G-weighted sum of sy
    float *part_p, *part_g;      // split > 1: their fp32 partial sums [split][bh][n_f][64]
    // partial maxima of |sg|, |sy| ([kMaxParts][64] per head, heads 4 kMaxParts 64 apart), or null: scanned
    const float *max_g, *max_y;
    const float *tmax_g, *tmax_y;  // beside them: of each kTileRows-row tile ([kFineTiles] per head), n_s <= kFineRows
    int n_f, n_s;
};

struct TileArgs {
    TileSide side[2];
    int64_t bh;
    int sides, m, tau;
    int parts;  // row ranges that have maxima (of the kMaxParts of a head), where there are any
    int split;  // workgroups per block of fixed rows, each streaming a contiguous share
    float pbase, pinv;  // YOSO-E: p = (base pbase)^tau, 1 / pbase^tau
};

// A constant the compiler does not see through: a multiply-add by it stays one, so that
// it can take an fp16 operand in place (v_fma_mix_f32) instead of converting it first.
__device__ __forceinline__ float opaque(float x) {
    asm("" : "+s"(x));
    return x;
}

// Lane l holds values of dims 8 (l mod 8) + [0, 8): their maxima over the wave's rows (every lane).
__device__ __forceinline__ void octet_max(float v[8]) {
#pragma unroll
    for (int i = 0; i < 8; i++) {
        float x = v[i];
        x = fmaxf(x, dpp_mov<0x128>(x));  // row_ror 8: lane l ^ 8
        const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        x = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
        const auto c = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
        v[i] = fmaxf(__uint_as_float(c[0]), __uint_as_float(c[1]));
    }
}
__device__ __forceinline__ void put_octet(float *row, int oct, const float v[8]) {
    reinterpret_cast<float4 *>(row + 8 * oct)[0] = make_float4(v[0], v[1], v[2], v[3]);
    reinterpret_cast<float4 *>(row + 8 * oct)[1] = make_float4(v[4], v[5], v[6], v[7]);
}

// The codes of both sides as bit planes [row][NW]: word t PW + w holds bit t of the codes
// of hashes 32 w .. 32 w + 31 (PW = 2 for NW = 16, else 1); words past tau PW and bits past
// m are zero.  One row per thread and word group w: the row's codes, 64 consecutive bytes,
// are read once; 2 operations per code and bit (4 us at 2 x 131072 rows of 32 8-bit codes,
// its traffic alone about 3).
// Blocks past the planes' (`plane_blocks`) take partial maxima instead: block (b*4 + t)
// parts + p writes the largest |x| of each of the 64 dims over the p-th of `parts` row ranges
// of tensor t (0 Q, 1 dY, 2 K, 3 V) of head b, from which the tiles derive their scales.  Up to
// kFineRows rows the ranges are whole tiles of kTileRows rows, whose largest |x| of all dims follows
// ([4 b + t][kFineTiles] after the parts of all heads).
template <int NW, bool BF16>
__global__ __launch_bounds__(256) void tile_prep_kernel(const uint16_t *__restrict__ qcodes,
                                                        const uint16_t *__restrict__ kcodes,
                                                        uint32_t *__restrict__ qpl, uint32_t *__restrict__ kpl,
                                                        int64_t rows_q, int64_t rows_k, int m, int tau,
                                                        int64_t plane_blocks, const void *__restrict__ q,
                                                        const void *__restrict__ dy, const void *__restrict__ k,
                                                        const void *__restrict__ v, int64_t n_q, int64_t n_k,
                                                        float *__restrict__ pmax, int parts, int fine_per) {
    constexpr int PW = NW == 16 ? 2 : 1, PT = NW / PW;  // planes stored per word group
    if (blockIdx.x >= plane_blocks) {
        const int64_t blk = blockIdx.x - plane_blocks, bt = blk / parts;
        const int p = static_cast<int>(blk - bt * parts), t = static_cast<int>(bt) & 3;
        const int64_t b = bt >> 2, heads4 = (gridDim.x - plane_blocks) / parts;
        float *dst = pmax + (bt * kMaxParts + p) * D;
        const void *src = t == 0 ? q : t == 1 ? dy : t == 2 ? k : v;
        const int64_t n = t < 2 ? n_q : n_k;
        // (up to kFineRows rows: `fine_per` per block, one to four tiles of 32, each one step of the block)
        static_assert(kFineRows == kMaxParts * 4 * kTileRows && kTileRows == 32, "");
        const bool fine = n <= kFineRows;
        const int64_t per = fine ? fine_per : (n + kMaxParts - 1) / kMaxParts;
        const int64_t r0 = min(n, p * per), r1 = min(n, r0 + per);
        const int d = threadIdx.x;
        if (r0 == r1) {
            if (d < D) dst[d] = 0.f;
            return;
        }
        const int64_t base = (b * n + r0) * D, count = (r1 - r0) * D;
        __shared__ __align__(16) float wred[4][D];
        __shared__ float tred[4][4];
        float mx[8] = {};   // (a thread keeps to dims 8 (t mod 8) + [0, 8))
        float tmx[4] = {};  // its rows of the four tiles
        for (int64_t e0 = static_cast<int64_t>(threadIdx.x) * 8; e0 < count; e0 += 256 * 8 * 4) {
            float x[4][8];
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int64_t e = e0 + u * 256 * 8;
                load8<BF16>(src, base + (e < count ? e : e0), x[u]);  // (past the end: this thread's first again)
            }
#pragma unroll
            for (int u = 0; u < 4; u++) {
                float w = 0.f;
#pragma unroll
                for (int i = 0; i < 8; i++) {
                    mx[i] = fmaxf(mx[i], fabsf(x[u][i]));
                    w = fmaxf(w, fabsf(x[u][i]));
                }
                if (fine) tmx[u] = e0 + u * 256 * 8 < count ? w : 0.f;
            }
        }
        if (fine) {
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const float w = wave_max(tmx[u]);
                if ((threadIdx.x & 63) == 0) tred[u][threadIdx.x >> 6] = w;
            }
        }
        octet_max(mx);
        if ((threadIdx.x & 63) < 8) put_octet(wred[threadIdx.x >> 6], threadIdx.x & 7, mx);
        __syncthreads();
        if (d < D) dst[d] = fmaxf(fmaxf(wred[0][d], wred[1][d]), fmaxf(wred[2][d], wred[3][d]));
        const int64_t tile = r0 / kTileRows + d;
        if (fine && d < 4 && tile * kTileRows < r1)
            pmax[heads4 * (kMaxParts * D) + bt * kFineTiles + tile] =
                fmaxf(fmaxf(tred[d][0], tred[d][1]), fmaxf(tred[d][2], tred[d][3]));
        return;
    }
    const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    const int64_t total = (rows_q + rows_k) * PW;
    if (t >= total) return;
    const int64_t r = t / PW;
    const int w = static_cast<int>(t - r * PW);
    const bool kside = r >= rows_q;
    const int64_t row = kside ? r - rows_q : r;
    const uint16_t *src = (kside ? kcodes : qcodes) + row * m + 32 * w;
    uint32_t *dst = (kside ? kpl : qpl) + row * NW + w;
    const int valid = min(32, m - 32 * w);
    uint32_t pl[PT];
#pragma unroll
    for (int j = 0; j < PT; j++) pl[j] = 0u;
    if (valid == 32 && (m & 7) == 0) {  // (codes are 16-byte aligned)
#pragma unroll
        for (int v = 0; v < 4; v++) {
            const uint4 c4 = reinterpret_cast<const uint4 *>(src)[v];
            const uint32_t c[4] = {c4.x, c4.y, c4.z, c4.w};
#pragma unroll
            for (int i = 0; i < 4; i++)
#pragma unroll
                for (int j = 0; j < PT; j++) {
                    pl[j] |= __builtin_amdgcn_ubfe(c[i], j, 1) << (8 * v + 2 * i);
                    pl[j] |= __builtin_amdgcn_ubfe(c[i], 16 + j, 1) << (8 * v + 2 * i + 1);
                }
        }
    } else {
        for (int h = 0; h < valid; h++) {
            const uint32_t c = src[h];
#pragma unroll
            for (int j = 0; j < PT; j++) pl[j] |= ((c >> j) & 1u) << h;
        }
    }
#pragma unroll
    for (int j = 0; j < PT; j++) dst[j * PW] = j < tau ? pl[j] : 0u;  // (bits of a code past tau are not part of it)
}

// One plane word of a row from the codes of its word group (four groups of eight codes;
// those past m read as zeros): bit h of the word is bit t of code h.
__device__ __forceinline__ uint32_t plane_word(const uint4 c[4], int t) {
    uint32_t w = 0u;
#pragma unroll
    for (int v = 0; v < 4; v++) {
        const uint32_t x[4] = {c[v].x, c[v].y, c[v].z, c[v].w};
#pragma unroll
        for (int i = 0; i < 4; i++) {
            w |= __builtin_amdgcn_ubfe(x[i], t, 1) << (8 * v + 2 * i);
            w |= __builtin_amdgcn_ubfe(x[i], 16 + t, 1) << (8 * v + 2 * i + 1);
        }
    }
    return w;
}
// the codes of hashes 32 w .. of a row (m a multiple of 8, codes 16-byte aligned)
__device__ __forceinline__ void load_group(uint4 c[4], const uint16_t *row, int m, int w) {
#pragma unroll
    for (int v = 0; v < 4; v++) {
        const bool in = 32 * w + 8 * v < m;
        c[v] = *reinterpret_cast<const uint4 *>(row + (in ? 32 * w + 8 * v : 0));
        const uint32_t keep = in ? 0xFFFFFFFFu : 0u;
        c[v].x &= keep; c[v].y &= keep; c[v].z &= keep; c[v].w &= keep;
    }
}

// hi, lo of v * scale (scale a power of two, or the product rounded once in fp32)
__device__ __forceinline__ void split8_pk(const float v[8], float scale, half8 &hi, half8 &lo) {
#pragma clang fp contract(off)
    const float mone = opaque(-1.0f);
#pragma unroll
    for (int i = 0; i < 8; i += 2) {
        float a = v[i] * scale, b = v[i + 1] * scale;
        asm volatile("" : "+v"(a), "+v"(b));
        const half2v h = __builtin_convertvector(float2v{a, b}, half2v);
        const half2v l = __builtin_convertvector(float2v{fmaf(static_cast<float>(h[0]), mone, a),
                                                         fmaf(static_cast<float>(h[1]), mone, b)}, half2v);
        hi[i] = h[0]; hi[i + 1] = h[1];
        lo[i] = l[0]; lo[i + 1] = l[1];
    }
}

// LDS by byte address.  A lane base is made opaque, so that it stays one register and the
// constants added to it become instruction offsets.
typedef __attribute__((address_space(3))) unsigned char *lds_bytes;
__device__ __forceinline__ uint32_t lane_base(uint32_t a) {
    asm("" : "+v"(a));
    return a;
}
template <typename T>
__device__ __forceinline__ T lds_get(uint32_t a) {
    return *reinterpret_cast<const __attribute__((address_space(3))) T *>(a);
}
template <typename T>
__device__ __forceinline__ void lds_put(uint32_t a, const T &v) {
    *reinterpret_cast<__attribute__((address_space(3))) T *>(a) = v;
}

// Streamed tiles: rows of 256 bytes [hi 64 | lo 64], 16-byte chunk c of row r at slot
// c ^ f(r).  f is a bijection of r mod 16, so that 16 rows read at one chunk hit distinct
// banks, and f >> 2 differs within every 4 aligned rows, so that a transposing read (4
// rows x 4 chunks per half-wave) does too.
__device__ __forceinline__ uint32_t tswz(int row) {
    return static_cast<uint32_t>(((row & 3) << 2) | ((row >> 2) & 3));
}

__device__ __forceinline__ half4 tile_tr(uint32_t a) {
    typedef short short4v __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) short4v lds_short4;
    return __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)(static_cast<uintptr_t>(a))));
}

__device__ __forceinline__ floatx16 mfma32(const half8 &a, const half8 &b, const floatx16 &c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// x^n by squarings and multiplications
template <int N>
__device__ __forceinline__ float ipow(float x) {
    if constexpr (N == 1) return x;
    else {
        const float h = ipow<N / 2>(x);
        return N % 2 ? h * h * x : h * h;
    }
}
template <int N>
__device__ __forceinline__ void ipow16(floatx16 &p) {
#pragma unroll
    for (int i = 0; i < 16; i++) p[i] = ipow<N>(p[i]);
}

// scale_exp for the norm of a row held as 32 values each by lanes l and l ^ 32.  (The squares of
// rows of any finite size overflow or vanish; those of rows scaled by their largest value
// do not.)
__device__ __forceinline__ int norm_exp(const float v[4][8]) {
    float mx = 0.f;
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int i = 0; i < 8; i++) mx = fmaxf(mx, fabsf(v[s][i]));
    const int e0 = scale_exp(fmaxf(mx, __shfl_xor(mx, 32)));
    const float sc = ldexpf(1.0f, -e0);
    float ss = 0.f;
#pragma unroll
    for (int s = 0; s < 4; s++)
#pragma unroll
        for (int i = 0; i < 8; i++) ss = fmaf(v[s][i] * sc, v[s][i] * sc, ss);
    ss += __shfl_xor(ss, 32);
    int e2 = 0;
    if (ss > 0.f) frexpf(ss, &e2);  // ss < 2^e2: the norm is below 2^(e0 + ceil(e2/2))
    return e0 + ((e2 + 1) >> 1);
}

// 8 values of a row as loaded
template <bool BF16>
struct Raw {
    uint4 w[BF16 ? 1 : 2];
};
template <bool BF16>
__device__ __forceinline__ void raw_load(Raw<BF16> &r, const void *base, int64_t off) {
    const uint4 *p = reinterpret_cast<const uint4 *>(static_cast<const char *>(base) + off * (BF16 ? 2 : 4));
    r.w[0] = p[0];
    if constexpr (!BF16) r.w[1] = p[1];
}
template <bool BF16>
__device__ __forceinline__ void raw_values(const Raw<BF16> &r, float v[8]) {
    const uint32_t a[4] = {r.w[0].x, r.w[0].y, r.w[0].z, r.w[0].w};
    if constexpr (BF16) {
#pragma unroll
        for (int i = 0; i < 4; i++) {
            v[2 * i] = __uint_as_float(a[i] << 16);
            v[2 * i + 1] = __uint_as_float(a[i] & 0xFFFF0000u);
        }
    } else {
        const uint32_t b[4] = {r.w[1].x, r.w[1].y, r.w[1].z, r.w[1].w};
#pragma unroll
        for (int i = 0; i < 4; i++) {
            v[i] = __uint_as_float(a[i]);
            v[4 + i] = __uint_as_float(b[i]);
        }
    }
}

// LDS bytes of a workgroup: the double-buffered tiles and counts
template <int WT, int SUM, int NW, int WAVES>
constexpr int tile_lds() {
    constexpr int T = 8 * WAVES;
    constexpr int tiles = 1 + (SUM != kSumP ? 1 : 0) + (WT == kWeightExpect ? 1 : 0);
    constexpr int counts = WT == kWeightExpect ? 0 : 32 * WAVES * T * 2 + T * NW * 4;
    return 2 * (tiles * T * 256 + counts);
}

// Waves per SIMD that the registers are cut for: two; three for the bf16 forms that need at
// most 168 (64 x 1500 x 1030 backward: 226 -> 216 us, 192 x 1500 forward: 323 -> 283)
template <int WT, int SUM, bool BF16, int NW>
constexpr int kWavesPerSimd = WT == kWeightCount && SUM != kSumPG && BF16 && NW == 8 ? 3 : 2;

// NW: plane words per row (8: tau <= 8; 12: tau <= 12; 16: two words per plane, tau <= 8)
template <int WT, int SUM, bool BF16, int NW, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((
    amdgpu_waves_per_eu(kWavesPerSimd<WT, SUM, BF16, NW>, kWavesPerSimd<WT, SUM, BF16, NW>))) void tile_kernel(TileArgs args) {
    constexpr bool kP = SUM != kSumG, kG = SUM != kSumP;
    constexpr bool kExp = WT == kWeightExpect, kStar = WT == kWeightStar;
    constexpr bool kX = WT != kWeightCount;  // a scalar product x beside G
    constexpr bool kRowScale = kStar;        // weights scaled per fixed row as they come
    constexpr bool kCountG = kG && !kX;      // G weighted by counts
    constexpr bool kFlush = kCountG && !BF16 && (NW != 12 || !kP);  // long sums in parts of kFlushRows rows
    constexpr int kFE = kCountG ? kFixedExpCount : kFixedExp;
    // the rows that counts alone weight (dV's dY, the forward's V) are scaled dim by dim
    constexpr bool kDims = kP && !kX;
    constexpr bool kFine = !kStar;  // tiles may have scales of their own
    constexpr bool kOwnPlanes = !kExp && !kG;  // the forward: planes built here from the codes
    constexpr int PW = NW == 16 ? 2 : 1;       // word groups of 32 hashes
    constexpr int T = 8 * WAVES;             // streamed rows per tile
    constexpr int NB = T / 32;               // 32-row blocks per tile
    constexpr int TB = T * 256;              // LDS bytes of one tensor's tile
    constexpr int kTiles = 1 + (kG ? 1 : 0) + (kExp ? 1 : 0);
    constexpr int CROW = T * 2;              // LDS bytes of a fixed row's counts
    constexpr int CB = kExp ? 0 : 32 * WAVES * CROW;
    constexpr int PB = kExp ? 0 : T * NW * 4;  // the streamed rows' plane words
    // LDS: the two buffers of each kind side by side (cosine rows, rows of G, summed rows,
    // counts, planes), so that an access class reaches all it uses from one lane base within
    // the 16-bit offsets of the LDS instructions
    constexpr int OX0 = 0, OG = kExp ? 2 * TB : 0, OY = OG + (kG ? 2 * TB : 0), OX = kStar ? OY : OX0;
    constexpr int OC = OY + 2 * TB, OP = OC + 2 * CB;
    constexpr int OSUM = kP && kG ? OG : OY;  // the first rows that sums read
    // a word per tile of each streamed tensor, sy, then sg (counts: of up to kFineRows rows)
    constexpr int OT = kExp ? OY + 2 * TB : OP + 2 * PB;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float wmax[2][WAVES];
    __shared__ int wfar[WAVES];  // a tile far below its head
    __shared__ __align__(16) float dmax[kDims ? WAVES : 1][D];  // the waves' maxima per dim
    __shared__ __align__(16) float dscale[kDims ? D : 4];       // 2^(13 - e_d)
    __shared__ __align__(16) int dexp[kDims ? D : 4];           // e_d: the dim's |values| are below 2^e_d
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_bytes)smem));

    const int64_t t0 = (args.side[0].n_f + 32 * WAVES - 1) / (32 * WAVES);
    const int64_t t1 = args.sides > 1 ? (args.side[1].n_f + 32 * WAVES - 1) / (32 * WAVES) : 0;
    const int split = args.split;
    const int64_t blk0 = xcd_remap(blockIdx.x, args.bh * (t0 + t1) * split);
    const int sp = static_cast<int>(blk0 % split);
    const int64_t blk = blk0 / split;
    const bool second = blk >= args.bh * t0;
    const TileSide a = args.side[second ? 1 : 0];
    const int64_t lblk = second ? blk - args.bh * t0 : blk;
    const int64_t tf = second ? t1 : t0;
    const int64_t b = lblk / tf;
    const int r0 = static_cast<int>(lblk - b * tf) * (32 * WAVES);
    const int nf = a.n_f, ns = a.n_s;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l31 = lane & 31, hh = lane >> 5;
    // streamed rows [cs0, cs1) of this workgroup, whole tiles
    const int slen = ((ns + split - 1) / split + T - 1) / T * T;
    const int cs0 = min(ns, sp * slen), cs1 = min(ns, cs0 + slen);

    // ---- staging role: thread t stages 8 dims (16-byte chunk) of row t / 8 of a tile
    const int srow = tid >> 3, soct = tid & 7;
    const int64_t sbase = b * ns * D + 8 * soct;
    // (the tensors of a tile are loaded and staged one after another through one set of
    // registers: part 0 the summed rows, 1 the rows of G or else the cosine rows, 2 the cosine rows)
    Raw<BF16> raw;
    constexpr int kParts = kTiles;
    constexpr int kPlaneThreads = T * NW / 4;  // threads that stage 4 plane words each
    uint4 rp;
    uint4 rcodes[4];  // (forward: thread t builds words t % 8 and t % 8 + 8 of row t / 8 of a tile)
    auto load_planes = [&](int c0) {
        if constexpr (kOwnPlanes) {
            load_group(rcodes, a.scodes + (b * ns + min(c0 + srow, ns - 1)) * args.m, args.m, soct & (PW - 1));
        } else if constexpr (!kExp) {
            const int e = min(tid, kPlaneThreads - 1), r = e / (NW / 4);
            rp = reinterpret_cast<const uint4 *>(a.spl + (b * ns + min(c0 + r, ns - 1)) * NW)[e - r * (NW / 4)];
        }
    };
    auto load_part = [&](int c0, int part) {
        const int64_t off = sbase + static_cast<int64_t>(min(c0 + srow, ns - 1)) * D;
        raw_load<BF16>(raw, part == 0 ? a.sy : kG && part == 1 ? a.sg : a.sx, off);
    };

    // ---- the streamed tensors' largest |value| over the head (every split scans all of
    // it, so that the scales, and the results, do not depend on the share)
    float mg = 0.f, my = 0.f, md[8] = {};
    const bool have_max = a.max_y != nullptr;
    // of each tile of T rows, too (words at OT); a wave scans 64 rows at a time
    const bool fine = kExp || (kFine && ns <= kFineRows);
    const int ntiles = fine ? (ns + T - 1) / T : 0;
    const int nwords = kExp ? ntiles : kFineTiles;
    if (kFine && fine && !have_max) {
        for (int g0 = 64 * wave; g0 < ns; g0 += 64 * WAVES) {
            Raw<BF16> u[8], w[8];
#pragma unroll
            for (int i = 0; i < 8; i++) {
                const int64_t off = (b * ns + min(g0 + 8 * i + (lane >> 3), ns - 1)) * D + 8 * (lane & 7);
                raw_load<BF16>(u[i], a.sy, off);
                if constexpr (kG) raw_load<BF16>(w[i], a.sg, off);
            }
#pragma unroll
            for (int h = 0; h < 64 / T; h++) {
                float ty = 0.f, tg = 0.f, td[8] = {};
#pragma unroll
                for (int i = h * (T / 8); i < (h + 1) * (T / 8); i++) {
                    float v[8];
                    raw_values<BF16>(u[i], v);
#pragma unroll
                    for (int e = 0; e < 8; e++) {
                        if constexpr (kDims && !kG) td[e] = fmaxf(td[e], fabsf(v[e]));
                        else ty = fmaxf(ty, fabsf(v[e]));
                    }
                    if constexpr (kG) {
                        raw_values<BF16>(w[i], v);
#pragma unroll
                        for (int e = 0; e < 8; e++) {
                            if constexpr (kDims) td[e] = fmaxf(td[e], fabsf(v[e]));
                            else tg = fmaxf(tg, fabsf(v[e]));
                        }
                    }
                }
                if constexpr (kDims) {
#pragma unroll
                    for (int e = 0; e < 8; e++) {
                        md[e] = fmaxf(md[e], td[e]);
                        if constexpr (kG) tg = fmaxf(tg, td[e]);
                        else ty = fmaxf(ty, td[e]);
                    }
                }
                ty = wave_max(ty);
                if constexpr (kG) tg = wave_max(tg);
                const int tile = g0 / T + h;
                if (lane == 0 && tile < ntiles) {
                    lds_put<float>(lds0 + OT + 4 * tile, ty);
                    if constexpr (kG) lds_put<float>(lds0 + OT + 4 * (nwords + tile), tg);
                }
                my = fmaxf(my, ty);
                mg = fmaxf(mg, tg);
            }
        }
    }
    if (have_max) {
        // (lane: dims 8 (lane mod 8) + [0, 8) of part lane / 8; of the last where there are fewer)
        static_assert(kMaxParts == 8, "a part per eight lanes");
        const int64_t e = (b * 4 * kMaxParts + min(lane >> 3, args.parts - 1)) * D + 8 * (lane & 7);
#pragma unroll
        for (int i = 0; i < 8; i++) {
            my = fmaxf(my, a.max_y[e + i]);
            if constexpr (kG) mg = fmaxf(mg, a.max_g[e + i]);
        }
        if constexpr (kDims) {
            const float *src = kG ? a.max_g : a.max_y;
#pragma unroll
            for (int i = 0; i < 8; i++) md[i] = src[e + i];
        }
        if (kFine && tid < ntiles) {
            auto tile_max = [&](const float *t, int to) {
                const float *w = t + b * (4 * kFineTiles) + tid * (T / kTileRows);
                float m = w[0];
                if (T > kTileRows && tid * T + kTileRows < ns) m = fmaxf(m, w[1]);
                lds_put<float>(lds0 + OT + 4 * to, m);
            };
            tile_max(a.tmax_y, tid);
            if constexpr (kG) tile_max(a.tmax_g, nwords + tid);
        }
    }
    for (int c = have_max || fine ? ns : srow; c < ns; c += 4 * T) {
        Raw<BF16> u[4], w[4];
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int64_t off = sbase + static_cast<int64_t>(min(c + i * T, ns - 1)) * D;
            raw_load<BF16>(u[i], a.sy, off);
            if constexpr (kG) raw_load<BF16>(w[i], a.sg, off);
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            float v[8];
            raw_values<BF16>(u[i], v);
#pragma unroll
            for (int e = 0; e < 8; e++) {
                if constexpr (kDims && !kG) md[e] = fmaxf(md[e], fabsf(v[e]));
                else my = fmaxf(my, fabsf(v[e]));
            }
            if constexpr (kG) {
                raw_values<BF16>(w[i], v);
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    if constexpr (kDims) md[e] = fmaxf(md[e], fabsf(v[e]));
                    else mg = fmaxf(mg, fabsf(v[e]));
                }
            }
        }
    }
    load_part(cs0, 0);
    if constexpr (kDims) {
        octet_max(md);
        if (lane < 8) put_octet(dmax[wave], lane, md);
        float m = 0.f;
#pragma unroll
        for (int i = 0; i < 8; i++) m = fmaxf(m, md[i]);
        if constexpr (kG) mg = m;
        else my = m;
    }
    my = wave_max(my);
    if constexpr (kG) mg = wave_max(mg);
    if (lane == 0) {
        wmax[0][wave] = my;
        wmax[1][wave] = mg;
    }

    // ---- fixed rows as B operands: lane (l31, hh) holds row 32 wave + l31, dims 16 s + 8 hh + [0, 8)
    const int frow = r0 + 32 * wave + l31;
    const int64_t foff = (b * nf + min(frow, nf - 1)) * D + 8 * hh;
    half8 arh[4], arl[4], xrh[4], xrl[4];
    int ea = 0, ex = 0;
    float va[kG ? 4 : 1][8];
    auto fix_a = [&]() {
        if constexpr (kG) {
            ea = norm_exp(va);
#pragma unroll
            for (int s = 0; s < 4; s++) split8_pk(va[s], ldexpf(1.0f, kFE - ea), arh[s], arl[s]);
        }
    };
    if constexpr (kG) {
#pragma unroll
        for (int s = 0; s < 4; s++) load8<BF16>(a.fa, foff + 16 * s, va[s]);
        if constexpr (!kDims) fix_a();
    }
    if constexpr (kX) {
        float v[4][8];
#pragma unroll
        for (int s = 0; s < 4; s++) load8<BF16>(a.fx, foff + 16 * s, v[s]);
        float sc;
        if constexpr (kExp) {
            float ss = 0.f;
#pragma unroll
            for (int s = 0; s < 4; s++)
#pragma unroll
                for (int i = 0; i < 8; i++) ss = fmaf(v[s][i], v[s][i], ss);
            ss += __shfl_xor(ss, 32);
            sc = ss > 0.f ? kCosScale / sqrtf(ss) : 0.f;
        } else {
            ex = norm_exp(v);
            sc = ldexpf(1.0f, kFE - ex);
        }
#pragma unroll
        for (int s = 0; s < 4; s++) split8_pk(v[s], sc, xrh[s], xrl[s]);
    }

    // ---- counting role: lane = fixed rows 128 (wave mod WAVES/4) + lane and + 64 + lane,
    // partners T/4 (wave / (WAVES/4)) + [0, T/4) of a tile
    constexpr int QW = WAVES / 4;
    const int crow = 128 * (wave % QW) + lane, cpart = wave / QW;
    uint32_t qp[2][kExp ? 1 : NW];
    if constexpr (kOwnPlanes) {
        // the workgroup's fixed rows as planes, through the counts' space: thread t half of
        // the words of row t / 2
        const int row = tid >> 1, half = tid & 1;
        uint4 c[4];
        load_group(c, a.fcodes + (b * nf + min(r0 + row, nf - 1)) * args.m, args.m, PW == 2 ? half : 0);
#pragma unroll
        for (int i = 0; i < NW / 2; i++) {
            const int t = PW == 2 ? i : (NW / 2) * half + i;
            lds_put<uint32_t>(lds0 + OC + row * (NW * 4) + 4 * (PW == 2 ? 2 * i + half : t),
                              t < args.tau ? plane_word(c, t) : 0u);
        }
        __syncthreads();
    }
    if constexpr (!kExp) {
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const uint4 *src =
                reinterpret_cast<const uint4 *>(a.fpl + (b * nf + min(r0 + crow + 64 * r, nf - 1)) * NW);
#pragma unroll
            for (int j = 0; j < NW / 4; j++) {
                uint4 w4;
                if constexpr (kOwnPlanes) {
                    const u32x4 x = lds_get<u32x4>(lds0 + OC + (crow + 64 * r) * (NW * 4) + 16 * j);
                    w4 = make_uint4(x[0], x[1], x[2], x[3]);
                } else {
                    w4 = src[j];
                }
                qp[r][4 * j] = w4.x; qp[r][4 * j + 1] = w4.y; qp[r][4 * j + 2] = w4.z; qp[r][4 * j + 3] = w4.w;
            }
        }
    }
    // C is kept as C 2^-11 (an exact fp16 number; *YOSO keeps N itself and scales the weight)
    constexpr float cscale = 1.0f / (1 << kCountExp);

    __syncthreads();
    float hy = 0.f, hg = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; w++) {
        hy = fmaxf(hy, wmax[0][w]);
        hg = fmaxf(hg, wmax[1][w]);
    }
    const int ey = __builtin_amdgcn_readfirstlane(scale_exp(hy));
    const int eg = kG ? __builtin_amdgcn_readfirstlane(scale_exp(hg)) : 0;
    const float scy = ldexpf(1.0f, 13 - ey), scg = ldexpf(1.0f, 13 - eg);
    // The exponents of the tiles.  A tile keeps its head's until its largest value is 2^8
    // below (then it has 30 bits left above the pairs' end), and follows it down to 2^40.  (Counts:
    // up to kFineRows rows.)
    bool varied = false;  // (no tile has: nothing of this in the loop)
    if (kFine && ntiles > 0) {
        bool far = false;
        for (int i = tid; i < (kG ? 2 : 1) * ntiles; i += 64 * WAVES) {
            const bool y = i < ntiles;
            const int at = lds0 + OT + 4 * (y ? i : nwords + i - ntiles);
            const float m = lds_get<float>(at);
            const int head = y ? ey : eg, e = m > 0.f ? scale_exp(m) : head;
            far = far || e < head - 8;
            lds_put<int>(at, e < head - 8 ? max(e, head - 40) : head);
        }
        const bool any = __builtin_amdgcn_ballot_w64(far) != 0;
        if (lane == 0) wfar[wave] = any ? 1 : 0;
    }
    if constexpr (kDims) {
        if (tid < D) {
            float m = 0.f;
#pragma unroll
            for (int w = 0; w < WAVES; w++) m = fmaxf(m, dmax[w][tid]);
            const int e = m > 0.f ? scale_exp(m) : -100;  // (a dim of zeros: nothing of a)
            dscale[tid] = ldexpf(1.0f, 13 - e);
            dexp[tid] = e;
        }
    }
    if (kDims || (kFine && ntiles > 0)) __syncthreads();
    if (kFine && ntiles > 0) {
        int f = 0;
#pragma unroll
        for (int w = 0; w < WAVES; w++) f |= wfar[w];
        varied = __builtin_amdgcn_readfirstlane(f) != 0;
    }
    auto tile_y = [&](int c0) { return lds_get<int>(lds0 + OT + 4 * (c0 / T)); };
    auto tile_g = [&](int c0) { return lds_get<int>(lds0 + OT + 4 * (nwords + c0 / T)); };
    if constexpr (kDims) {
        // A tile of rows scaled dim by dim follows the dim that lies least below its own of the head
        if (varied) {
            constexpr int to = OT + (kG ? 4 * kFineTiles : 0);
            const int head = kG ? eg : ey;
            for (int t = wave; t < ntiles; t += WAVES) {
                if (lds_get<int>(lds0 + to + 4 * t) == head) continue;  // (its largest value is not far below)
                float m[8] = {};
                for (int i = 0; i < T / 8; i++) {
                    const int64_t off = (b * ns + min(t * T + 8 * i + (lane >> 3), ns - 1)) * D + 8 * (lane & 7);
                    Raw<BF16> u;
                    raw_load<BF16>(u, kG ? a.sg : a.sy, off);
                    float v[8];
                    raw_values<BF16>(u, v);
#pragma unroll
                    for (int e = 0; e < 8; e++) m[e] = fmaxf(m[e], fabsf(v[e]));
                }
                octet_max(m);
                float above = -40.f;
#pragma unroll
                for (int e = 0; e < 8; e++)
                    if (m[e] > 0.f) above = fmaxf(above, static_cast<float>(scale_exp(m[e]) - dexp[8 * (lane & 7) + e]));
                const int d = static_cast<int>(wave_max(above + 64.f)) - 64;
                if (lane == 0) lds_put<int>(lds0 + to + 4 * t, d < -8 ? head + d : head);
            }
            __syncthreads();
        }
        // G = a . g: what scales a dim of g is taken back from a (up to the head's power)
        if constexpr (kG) {
#pragma unroll
            for (int s = 0; s < 4; s++)
#pragma unroll
                for (int i = 0; i < 8; i++) va[s][i] = ldexpf(va[s][i], dexp[16 * s + 8 * hh + i] - eg);
            fix_a();
        }
    }

    // the scales of the tile that is staged (of rows scaled dim by dim: beside those)
    float sty = kDims && !kG ? 1.0f : scy, stg = kDims ? 1.0f : scg;
    auto stage_scales = [&](int c0) {
        sty = ldexpf(1.0f, (kDims && !kG ? ey : 13) - __builtin_amdgcn_readfirstlane(tile_y(c0)));
        if constexpr (kG) stg = ldexpf(1.0f, (kDims ? eg : 13) - __builtin_amdgcn_readfirstlane(tile_g(c0)));
    };

    // convert and stage the tensor held in the raw registers (rows past cs1 as zeros)
    const uint32_t st_h = lane_base(lds0 + srow * 256 + ((soct ^ tswz(srow)) << 4));
    const uint32_t st_l = lane_base(lds0 + srow * 256 + (((8 + soct) ^ tswz(srow)) << 4));
    auto stage = [&](int bi, int c0, int part) {
        const bool ok = c0 + srow < cs1;
        auto put = [&](uint32_t t, const Raw<BF16> &r, float scale, bool lo_too, bool unit) {
            float v[8];
            raw_values<BF16>(r, v);
            if (unit) {
                float ss = 0.f;
#pragma unroll
                for (int i = 0; i < 8; i++) ss = fmaf(v[i], v[i], ss);
                ss = group_sum(ss, 8);  // the row's 8 threads
                scale = ss > 0.f ? kCosScale / sqrtf(ss) : 0.f;
            }
            half8 h, l;
            split8_pk(v, ok ? scale : 0.f, h, l);
            lds_put<half8>(st_h + t, h);
            if (lo_too) lds_put<half8>(st_l + t, l);
        };
        auto put_dims = [&](uint32_t t) {
            float v[8];
            raw_values<BF16>(raw, v);
            const float *sc = dscale + 8 * soct;
            const float4 s0 = reinterpret_cast<const float4 *>(sc)[0], s1 = reinterpret_cast<const float4 *>(sc)[1];
            v[0] *= s0.x; v[1] *= s0.y; v[2] *= s0.z; v[3] *= s0.w;
            v[4] *= s1.x; v[5] *= s1.y; v[6] *= s1.z; v[7] *= s1.w;
            half8 h, l;
            split8_pk(v, ok ? (kG ? stg : sty) : 0.f, h, l);
            lds_put<half8>(st_h + t, h);
            if (!BF16) lds_put<half8>(st_l + t, l);
        };
        if (kDims && !kG) put_dims(OY + bi * TB);
        else if (part == 0) put(OY + bi * TB, raw, sty, !BF16, false);
        else if (kDims && part == 1) put_dims(OG + bi * TB);
        else if (kG && part == 1) put(OG + bi * TB, raw, stg, !BF16, false);
        else put(OX + bi * TB, raw, 1.0f, true, true);
    };

    const uint32_t pl_w = lds0 + OP + tid * 16;
    const uint32_t pw_w = lds0 + OP + srow * (NW * 4) + soct * 4;
    auto stage_planes = [&](int bi) {
        if constexpr (kOwnPlanes) {
#pragma unroll
            for (int i = 0; i < 2; i++) {
                const int j = soct + 8 * i, t = j / PW;
                if (8 * i < NW && j < NW)
                    lds_put<uint32_t>(pw_w + bi * PB + 32 * i, t < args.tau ? plane_word(rcodes, t) : 0u);
            }
        } else if constexpr (!kExp) {
            if (tid < kPlaneThreads) lds_put<u32x4>(pl_w + bi * PB, u32x4{rp.x, rp.y, rp.z, rp.w});
        }
    };

    // Counting in slices of one partner and the lane's two fixed rows, woven between the
    // MFMAs of the tile before.  The partner's plane words come from LDS, the same for all
    // lanes.  (As scalar loads they cost more: a vector instruction with a scalar operand
    // takes 4.4 clocks of a SIMD shared by two waves, the all-vector v_bitop3 2.55.)
    // Partners in the order of the chunks that hold their counts: slice j takes partner
    // 8 (e / 4) + 4 g + e % 4 of the group of 16, e = j % 8, g = (j / 8) % 2.
    constexpr int NSL = T / 4;  // slices per tile
    struct Words {
        u32x4 w[NW / 4];
    };
    const uint32_t pl_r = lane_base(lds0 + OP + (T == 64 ? 16 * cpart : 16 * (cpart >> 1) + 4 * (cpart & 1)) * (NW * 4));
    auto load_words = [&](Words &d, int bi, int j) {
        if constexpr (!kExp) {
            // (T / 4 is 16 or 8 partners: a whole group of 16, or its half g = cpart & 1)
            const int e = j & 7;
            const int r = 8 * (e >> 2) + 4 * (j >> 3) + (e & 3);
#pragma unroll
            for (int i = 0; i < NW / 4; i++) d.w[i] = lds_get<u32x4>(pl_r + bi * PB + r * (NW * 4) + 16 * i);
        }
    };
    auto count_one = [&](const uint32_t *q, const Words &ws) -> uint32_t {
        uint32_t d[2] = {0u, 0u}, d2[2] = {0u, 0u};
#pragma unroll
        for (int j = 0; j < NW; j++) {
            const int z = NW == 16 ? j & 1 : 0;
            const uint32_t w = ws.w[j / 4][j % 4];
            if constexpr (kStar)  // d2: the hashes with a second differing bit
                d2[z] = __builtin_amdgcn_bitop3_b32(d2[z], d[z], q[j] ^ w, 0xF8);
            d[z] = __builtin_amdgcn_bitop3_b32(d[z], q[j], w, 0xF6);  // d | (q ^ k)
        }
        const int e = __builtin_popcount(d[0]) + (NW == 16 ? __builtin_popcount(d[1]) : 0);
        // as an fp16 bit pattern: 1024 + k holds the integer k in its low bits
        if constexpr (kStar) {
            // tau (m - differing) + (differing in one bit only)
            const int one = __builtin_popcount(d[0] & ~d2[0]) + (NW == 16 ? __builtin_popcount(d[1] & ~d2[1]) : 0);
            return 0x6400u + static_cast<uint32_t>(args.tau * (args.m - e) + one);
        }
        return 0x6400u + static_cast<uint32_t>(e);
    };
    half2v c2[2][4];
    uint32_t ueven[2] = {0u, 0u};
    // (1024 + k) -> C 2^-11 = (m - k) csc, or N = k (*YOSO), in one exact fp16 multiply-add
    const float cm1 = kStar ? 1.0f : -cscale;
    const half2v cmul = {static_cast<_Float16>(cm1), static_cast<_Float16>(cm1)};
    const float ct1 = kStar ? -1024.0f : cscale * (1024.0f + static_cast<float>(args.m));
    const half2v cadd = {static_cast<_Float16>(ct1), static_cast<_Float16>(ct1)};
    // (rows crow and crow + 64 have one swizzle)
    const uint32_t cw_f = T == 64 ? (crow & 7) : ((crow >> 2) & 3);
    const uint32_t c_w0 = lane_base(lds0 + OC + crow * CROW + (((T == 64 ? 2 * cpart : cpart) ^ cw_f) << 4));
    const uint32_t c_w1 = lane_base(lds0 + OC + crow * CROW + (((2 * cpart + 1) ^ cw_f) << 4));
    // row r of slice j
    auto slice = [&](int bi, int j, const Words &w, int r) {
        if constexpr (!kExp) {
            const uint32_t u = count_one(qp[r], w);
            if ((j & 1) == 0) {
                ueven[r] = u;
                return;
            }
            const half2v c = __builtin_bit_cast(half2v, ueven[r] | (u << 16));
            c2[r][(j & 7) >> 1] = __builtin_elementwise_fma(c, cmul, cadd);
            if ((j & 7) == 7) {
                half8 h;
#pragma unroll
                for (int e = 0; e < 8; e++) h[e] = c2[r][e >> 1][e & 1];
                lds_put<half8>((j >> 3 ? c_w1 : c_w0) + bi * CB + 64 * r * CROW, h);
            }
        }
    };

    // ---- block products.  A operand of the scalar products: lane (l31, hh) = streamed row
    // 32 k + l31, dims 16 s + 8 hh + [0, 8)
    uint32_t ra[8];
#pragma unroll
    for (int i = 0; i < 8; i++)
        ra[i] = lane_base(lds0 + l31 * 256 + ((static_cast<uint32_t>(2 * i + hh) ^ tswz(l31)) << 4));
    auto rows_op = [&](int t, int k, int s, int lo) { return lds_get<half8>(ra[4 * lo + s] + t + 32 * k * 256); };
    // A operand of the sums: lane = dim 32 db + l31; element e of half hh is streamed row
    // 32 k + 16 s + 8 (e / 4) + 4 hh + e % 4, the rows whose weights register 8 s + e of the
    // lane's block result holds.  ds_read_b64_tr_b16 gives destination lane 4a+b of a 16-lane
    // group element b of the 8 bytes addressed by source lanes 4i+a (i = 0..3).
    const int l15 = lane & 15, ti = l15 >> 2, ta = l15 & 3, tg = (lane >> 4) & 1;
    uint32_t sa[4][2];
#pragma unroll
    for (int i = 0; i < 4; i++)
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int row = 4 * hh + ti + 8 * h;
            sa[i][h] = lane_base(lds0 + OSUM + row * 256 + 8 * (ta & 1) +
                                 ((static_cast<uint32_t>(4 * i + 2 * tg + (ta >> 1)) ^ tswz(row)) << 4));
        }
    auto sum_op = [&](int t, int k, int s, int db, int lo) {
        const int o = t - OSUM + (32 * k + 16 * s) * 256;
        const half4 x = tile_tr(sa[2 * lo + db][0] + o);
        const half4 y = tile_tr(sa[2 * lo + db][1] + o);
        return __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    const int cr = 32 * wave + l31;
    uint32_t ca_r[T / 16];
#pragma unroll
    for (int i = 0; i < T / 16; i++)
        ca_r[i] = lane_base(lds0 + OC + cr * CROW +
                            ((static_cast<uint32_t>(2 * i + hh) ^ (T == 64 ? (cr & 7) : ((cr >> 2) & 3))) << 4));
    floatx16 outp[2], outg[2];
#pragma unroll
    for (int db = 0; db < 2; db++)
#pragma unroll
        for (int i = 0; i < 16; i++) outp[db][i] = outg[db][i] = 0.f;

    // YOSO-E: p = (base pbase)^tau < 2^16, base = 1 - arccos(c)/pi.  Two polynomials, both
    // least squares at Chebyshev nodes.  Where every |c| of a block is at most 1/2 (almost
    // all blocks of unclustered rows): 1/2 + arcsin(c)/pi = 1/2 + c A(c^2), A of degree 5,
    // |error| < 7e-9.  Else, with u = 1 - |c|: arccos(|c|)/pi = sqrt(u) Q(u), Q of degree 7,
    // relative error 2e-8.
    const float bs = args.pbase;
    constexpr float sq = kCosScale * kCosScale;  // a block's S is c * sq
    float ca[6] = {0.31830987334251404f, 0.05305203050374985f, 0.023855842649936676f,
                   0.014495517127215862f, 0.007610586937516928f, 0.013545230962336063f};
    float cq[8] = {0.45015814900398254f, 0.037513915449380875f, 0.008425663225352764f, 0.00262420903891325f,
                   0.00044531628373079f, 0.0011004807893186808f, -0.0006614952581003308f, 0.0003937508736271411f};
    {
        float f = bs / sq;
#pragma unroll
        for (int i = 0; i < 6; i++) {
            ca[i] *= f;
            f /= sq * sq;
        }
#pragma unroll
        for (int i = 0; i < 8; i++) cq[i] *= bs;
    }
    // W = G P 2^-7: |G| < 2^22, P <= 1
    const float wp = ldexpf(args.pinv, -7);
    // *YOSO: x = S 2^(ex - 6) 2^(ey - 13); weight (s / pi) / sqrt(max(1 - x^2, 1/64)), at most s 2.55
    const float xs = kStar ? ldexpf(1.0f, ex - kFE + ey - 13) : 0.f;
    const float sw = 0.31830988618379067f * ldexpf(1.0f, -kRowExp);

    // fp32 sums of a pair of halves are taken per block first (one of 32 dims at a time) and
    // then added to the running ones: an MFMA rounds its sum every 4 rows and there are three
    // per product, and that many roundings of the large sums cost precision (dQ at 4096
    // rows: error 6.0e-7 summed directly).  (YOSO-E's dK and dV have no registers for it; their
    // error is P's.  The backward's dV is summed directly too: its counts are exact, two products
    // per step at most.)
    constexpr bool kTwoLevel = !BF16 && !(kExp && kP && kG);

    // *YOSO: the lane's fixed row takes its weights times 2^-kw (fp32: of one block times 1 / unscale)
    int kw = 0;
    bool any_kw = false;  // some row of the wave has kw > 0
    float unscale = 1.0f;
    // Counts: |G| < 2^25, so the weight G C 2^-11 of up to three hashes stays below 2^16, and a
    // pair of one hash lies as high in the window as in the pair passes.  A row that meets a
    // count of 4 or more is scaled down by 2^2, from a count of 16 on by as much as m takes,
    // through its fixed row and with its running sums, before the tile's products.  The
    // exponent field of C 2^-11 is 4 for C = 1, 5 for 2 and 3, 6 or 7 for 4 to 15, 8 to 10 from
    // 16 on, so the bits of all counts of a row or'ed tell (`wmask`: those that ask for more).
    // (One scale for a count of m, 2^-12 at m = 32, left rows whose partners lie 10^4 below the
    // head's largest 4.8e-6 off in the median at 2048 rows, the pair passes 4.8e-7.)
    uint32_t wmask = 0x28002800u;
    auto count_kw = [&]() { return wmask == 0x28002800u ? 0 : wmask != 0 ? 2 : args.m < 64 ? 4 : 5; };
    auto widen = [&](int bi) {
        if constexpr (kCountG) {
            u32x4 o4 = lds_get<u32x4>(ca_r[0] + bi * CB);
#pragma unroll
            for (int i = 1; i < T / 16; i++) o4 |= lds_get<u32x4>(ca_r[i] + bi * CB);
            const uint32_t o = o4[0] | o4[1] | o4[2] | o4[3];
            if (__builtin_expect(__builtin_amdgcn_ballot_w64((o & wmask) != 0) == 0, 1)) return;
            // (the halves of the wave hold the same fixed rows)
            const auto r = __builtin_amdgcn_permlane32_swap(o, o, false, false);
            const uint32_t both = r[0] | r[1];
            const bool many = (both & 0x20002000u) != 0;
            const int k0 = count_kw(), k = (both & wmask) == 0 ? k0 : !many ? 2 : args.m < 64 ? 4 : 5;
            wmask = k == 0 ? 0x28002800u : k == 2 ? 0x20002000u : 0u;
            const float f = ldexpf(1.0f, k0 - k);
            const _Float16 fh = static_cast<_Float16>(f);
#pragma unroll
            for (int s = 0; s < 4; s++) {
                arh[s] *= fh;
                if constexpr (!BF16) arl[s] *= fh;
            }
#pragma unroll
            for (int db = 0; db < 2; db++) outg[db] *= f;
        }
    };

    const float zero = opaque(0.0f);
    auto split_w = [&](const float w[8], half8 &hi, half8 &lo) { split8_pk(w, 1.0f, hi, lo); };
    // *YOSO's weights of a block (`most`: the lane's largest) in the window of their pairs.  Where
    // the block's sums are taken apart (two levels), each row's are scaled by a power of two
    // of their own, which the sums take back as they are added.  Else the row's factor falls
    // when a weight would leave the window, and its running sums with it.
    auto row_scale = [&](float most, floatx16 &w) {
        if constexpr (!kTwoLevel) {
            if (__builtin_expect(!any_kw && __builtin_amdgcn_ballot_w64(most > kWeightMax) == 0, 1)) return;
        }
        // (the halves of the wave hold the same fixed rows)
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(most), __float_as_uint(most), false, false);
        const float row = fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
        int e = 0;
        if constexpr (kTwoLevel) {
            frexpf(row, &e);  // row < 2^e
            e = max(e - 15, -100);
            unscale = ldexpf(1.0f, e);
        } else {
            if (ldexpf(row, -kw) > kWeightMax) frexpf(row, &e);
            e = max(kw, e - 13);
            const float f = ldexpf(1.0f, kw - e);
#pragma unroll
            for (int db = 0; db < 2; db++) outg[db] *= f;
            kw = e;
            any_kw = __builtin_amdgcn_ballot_w64(kw > 0) != 0;
        }
        const float f = ldexpf(1.0f, -e);
#pragma unroll
        for (int i = 0; i < 16; i++) w[i] *= f;
    };

    // The products of a tile as a sequence of groups of one to three MFMAs on one operand
    // pair (hi, lo) from LDS: per block 4 groups of x and 4 of G (16 dims each), then 4 of the
    // P sum and 4 of the G sum (16 streamed rows, 32 dims each).  A group's operands are read
    // during the group before it.  x and G add their small products first, each of which rounds
    // the sum it finds (error of dQ at 1 x 512 1.64e-7, the large one first 1.70e-7; 1 x 64 1.42e-7
    // and 1.59e-7; the sums over rows gain nothing: 1 x 8192 2.52e-7 small first, 2.19e-7 large).
    // hook(i, 0), hook(i, 1), i = 0 .. 8 NB - 1, are called after the first and the last MFMA
    // of the groups that carry the next tile's work.
    struct Op {
        half8 h, l;
    };
    constexpr int kPX = kX ? 4 : 0, kPG = kG ? 4 : 0, kPP = kP ? 4 : 0;
    constexpr int kGroups = kPX + kPG + kPP + kPG;  // per block
    auto fetch = [&](int bi, int gi, Op &o) {
        const int k = gi / kGroups, i = gi % kGroups;
        if (i < kPX) {
            o.h = rows_op(OX + bi * TB, k, i, 0);
            if (kExp || !BF16) o.l = rows_op(OX + bi * TB, k, i, 1);
        } else if (i < kPX + kPG) {
            o.h = rows_op(OG + bi * TB, k, i - kPX, 0);
            if (!BF16) o.l = rows_op(OG + bi * TB, k, i - kPX, 1);
        } else {
            // (db, s) of the sums; the P sum (dV from dY, or the forward) first
            const int j = i - kPX - kPG;
            const bool psum = j < kPP;
            const int t = (psum && kG ? OG : OY) + bi * TB;
            const int sd = psum ? j : j - kPP;
            o.h = sum_op(t, k, sd & 1, sd >> 1, 0);
            if (!BF16) o.l = sum_op(t, k, sd & 1, sd >> 1, 1);
        }
    };
    auto compute = [&](int bi, auto hook) {
        Op op[2];
        // (beside the first operands' reads; where registers spill, before them: 51 -> 39 spills)
        constexpr bool kWidenFirst = NW == 16 && kP && !BF16;
        if (kWidenFirst) widen(bi);
        fetch(bi, 0, op[0]);
        if (!kWidenFirst) widen(bi);
        // group gi of the tile: `mm(j, o)` issues its j-th MFMA; hook index hi (or -1)
        auto group = [&](int gi, int n, int hi, auto mm) {
            const Op &o = op[gi & 1];
            mm(0, o);
            __builtin_amdgcn_sched_barrier(0);
            if (gi + 1 < kGroups * NB) fetch(bi, gi + 1, op[(gi + 1) & 1]);
            if (hi >= 0) hook(hi, 0);
            if (n > 1) mm(1, o);
            __builtin_amdgcn_sched_barrier(0);
            if (n > 2) mm(2, o);
            if (hi >= 0) hook(hi, 1);
        };
#pragma unroll
        for (int k = 0; k < NB; k++) {
            const int g0 = kGroups * k;
            floatx16 p, g;
#pragma unroll
            for (int i = 0; i < 16; i++) p[i] = g[i] = 0.f;
            if constexpr (kX) {
                constexpr int n = kExp || !BF16 ? 3 : 1;
#pragma unroll
                for (int s = 0; s < 4; s++)
                    group(g0 + s, n, kG ? -1 : 8 * k + s, [&](int j, const Op &o) {
                        p = mfma32(n == 3 && j == 1 ? o.l : o.h, n == 3 && j == 0 ? xrl[s] : xrh[s], p);
                    });
            }
            half8 c16[2];
            if constexpr (!kExp) {
#pragma unroll
                for (int s = 0; s < 2; s++) c16[s] = lds_get<half8>(ca_r[2 * k + s] + bi * CB);
            }
            if constexpr (kG) {
#pragma unroll
                for (int s = 0; s < 4; s++)
                    group(g0 + kPX + s, BF16 ? 1 : 3, 8 * k + s, [&](int j, const Op &o) {
                        g = mfma32(!BF16 && j == 1 ? o.l : o.h, !BF16 && j == 0 ? arl[s] : arh[s], g);
                    });
            }
            if constexpr (kExp) {
                float most = 0.f;
#pragma unroll
                for (int i = 0; i < 16; i += 2) most = fmaxf(fmaxf(most, fabsf(p[i])), fabsf(p[i + 1]));
                if (__builtin_amdgcn_ballot_w64(most > 0.5f * sq) == 0) {
#pragma unroll
                    for (int i = 0; i < 16; i++) {
                        const float z = p[i] * p[i];
                        float q = ca[5];
#pragma unroll
                        for (int j = 4; j >= 0; j--) q = fmaf(q, z, ca[j]);
                        p[i] = fmaf(p[i], q, 0.5f * bs);
                    }
                } else {
#pragma unroll
                    for (int i = 0; i < 16; i++) {
                        const float u = __saturatef(fmaf(-fabsf(p[i]), 1.0f / sq, 1.0f));
                        float q = cq[7];
#pragma unroll
                        for (int j = 6; j >= 0; j--) q = fmaf(q, u, cq[j]);
                        const float r = __builtin_amdgcn_sqrtf(u) * q;
                        p[i] = p[i] >= 0.f ? bs - r : r;
                    }
                }
                switch (args.tau) {  // (wave-uniform)
                    case 1: break;
                    case 2: ipow16<2>(p); break;
                    case 3: ipow16<3>(p); break;
                    case 4: ipow16<4>(p); break;
                    case 5: ipow16<5>(p); break;
                    case 6: ipow16<6>(p); break;
                    case 7: ipow16<7>(p); break;
                    case 8: ipow16<8>(p); break;
                    case 9: ipow16<9>(p); break;
                    case 10: ipow16<10>(p); break;
                    case 11: ipow16<11>(p); break;
                    default: ipow16<12>(p); break;
                }
            }
            // (hook0: the first of the hooks its four groups carry, `each` apiece, or -1)
            auto sums = [&](int gi0, int n, int hook0, int each, floatx16 (&out)[2], bool two, const half8 (&fh)[2],
                            const half8 (&fl)[2], bool pair) {
#pragma unroll
                for (int db = 0; db < 2; db++) {
                    floatx16 t;
                    if (two) {
#pragma unroll
                        for (int i = 0; i < 16; i++) t[i] = 0.f;
                    }
#pragma unroll
                    for (int s = 0; s < 2; s++) {
                        const int h = hook0 < 0 ? -1 : hook0 + each * (2 * db + s);
                        group(gi0 + 2 * db + s, n, h, [&](int j, const Op &o) {
                            floatx16 &acc = two ? t : out[db];
                            if (j == 0) acc = mfma32(o.h, fh[s], acc);
                            else if (pair && j == 1) acc = mfma32(o.h, fl[s], acc);
                            else acc = mfma32(o.l, fh[s], acc);
                        });
                        if (each == 2) {
                            hook(h + 1, 0);
                            hook(h + 1, 1);
                        }
                    }
                    if (two) {
                        if (kRowScale && n > 1 && &out == &outg) out[db] += t * unscale;
                        else out[db] += t;
                    }
                }
            };
            // P as a pair (C, exact, as hi alone); the forward, which has no G, carries the next
            // tile's work here
            if constexpr (kP) {
                half8 ph[2], pl[2];
#pragma unroll
                for (int s = 0; s < 2; s++) {
                    if constexpr (kExp) {
                        float w[8];
#pragma unroll
                        for (int e = 0; e < 8; e++) w[e] = p[8 * s + e];
                        split_w(w, ph[s], pl[s]);
                    } else {
                        ph[s] = pl[s] = c16[s];
                    }
                }
                sums(g0 + kPX + kPG, 1 + (kExp ? 1 : 0) + (BF16 ? 0 : 1), kG ? -1 : kX ? 8 * k + 4 : 8 * k,
                     kG || kX ? 1 : 2, outp, kTwoLevel && (kExp || !kG), ph, pl, kExp);
            }
            if constexpr (kG) {
#pragma unroll
                for (int i = 0; i < 16; i++) {
                    if constexpr (kExp) {
                        g[i] = g[i] * wp * p[i];
                    } else if constexpr (kStar) {
                        const float x = p[i] * xs;
                        const float z = fmaxf(fmaf(-x, x, 1.0f), kNearFloor);
                        g[i] *= static_cast<float>(c16[i >> 3][i & 7]) * (__builtin_amdgcn_rsqf(z) * sw);
                    } else {
                        g[i] = fmaf(g[i], static_cast<float>(c16[i >> 3][i & 7]), zero);
                    }
                }
                if constexpr (kRowScale) {
                    float most = 0.f;
#pragma unroll
                    for (int i = 0; i < 16; i += 2) most = fmaxf(fmaxf(most, fabsf(g[i])), fabsf(g[i + 1]));
                    row_scale(most, g);
                }
                half8 wh[2], wl[2];
#pragma unroll
                for (int s = 0; s < 2; s++) {
                    float w[8];
#pragma unroll
                    for (int e = 0; e < 8; e++) w[e] = g[8 * s + e];
                    split_w(w, wh[s], wl[s]);
                }
                sums(g0 + kPX + kPG + kPP, BF16 ? 2 : 3, 8 * k + 4, 1, outg, kTwoLevel, wh, wl, true);
            }
        }
    };

    int cy = ey, cg = eg;  // the exponents that the running sums are in

    // ---- outputs
    // (`again`: added to what a flush of the same sums has put there)
    auto finish = [&](bool again) {
        int row = tid;  // (frow again, not kept through the loop)
        if constexpr (kFlush) asm volatile("" : "+v"(row));
        const int h4 = (row >> 3) & 4;
        row = r0 + 32 * (row >> 6) + (row & 31);
        // o c 2^e (the power apart: it may pass the range of a scale where the output does not)
        auto put = [&](void *dst, float *part, const floatx16 o[2], float c, int e0, bool dims) {
#pragma unroll
            for (int db = 0; db < 2; db++)
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    // lane (l31, hh) holds out[row l31][32 db + 8 u + 4 hh + (0..3)] in registers 4u .. 4u+3
                    const int64_t off = (b * nf + row) * D + 32 * db + 8 * u + h4;
                    int4 e = make_int4(e0, e0, e0, e0);
                    if (dims) {
                        const int4 ed = reinterpret_cast<const int4 *>(dexp)[8 * db + 2 * u + h4 / 4];
                        e = make_int4(e0 + ed.x, e0 + ed.y, e0 + ed.z, e0 + ed.w);
                    }
                    float4 x = make_float4(ldexpf(o[db][4 * u] * c, e.x), ldexpf(o[db][4 * u + 1] * c, e.y),
                                                 ldexpf(o[db][4 * u + 2] * c, e.z), ldexpf(o[db][4 * u + 3] * c, e.w));
                    if (split > 1 || !BF16) {
                        float4 *to = reinterpret_cast<float4 *>(split > 1 ? part + sp * (args.bh * nf * D) + off
                                                                          : static_cast<float *>(dst) + off);
                        if (kFlush && again) {
                            const float4 y = *to;
                            x = make_float4(y.x + x.x, y.y + x.y, y.z + x.z, y.w + x.w);
                        }
                        *to = x;
                    } else {
                        uint2 w;
                        w.x = static_cast<uint32_t>(f32_to_bf16(x.x)) | (static_cast<uint32_t>(f32_to_bf16(x.y)) << 16);
                        w.y = static_cast<uint32_t>(f32_to_bf16(x.z)) | (static_cast<uint32_t>(f32_to_bf16(x.w)) << 16);
                        *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(dst) + off) = w;
                    }
                }
        };
        if (row < nf) {
            if constexpr (kP) {
                const int e1 = (kG ? cg : cy) - (kDims ? (kG ? eg : ey) : 0);
                // (the dQ side of a launch for both sides has no P output)
                if (a.out_p != nullptr)
                    put(a.out_p, a.part_p, outp, kExp ? args.pinv : 1.0f / static_cast<float>(args.m),
                        e1 - 13 + (kExp ? 0 : kCountExp), kDims);
            }
            if constexpr (kG) {
                const int e = (cg - 13) + (ea - kFE) + (cy - 13);
                const float half_tau = 0.5f * static_cast<float>(args.tau);
                if constexpr (kExp) put(a.out_g, a.part_g, outg, half_tau, e + 7, false);
                else if constexpr (kStar)
                    put(a.out_g, a.part_g, outg, 1.0f / static_cast<float>(args.m), e + kRowExp + kw, false);
                else put(a.out_g, a.part_g, outg, half_tau / static_cast<float>(args.m), e + kCountExp + count_kw(), false);
            }
        }
    };

    // ---- the pipeline: while tile t is computed, t + 1 is staged and counted and t + 2 loaded
    // (past the last tile the last one again, never used: no branch in the loop)
    const int clast = cs0 < cs1 ? cs0 + (cs1 - 1 - cs0) / T * T : cs0;
    if (cs0 < cs1) {
        load_planes(cs0);
        if (kFine && varied) stage_scales(cs0);
#pragma unroll
        for (int i = 0; i < kParts; i++) {
            if (i > 0) load_part(cs0, i);
            stage(0, cs0, i);
        }
        stage_planes(0);
        load_part(min(cs0 + T, clast), 0);
        load_planes(min(cs0 + T, clast));
    }
    if constexpr (!kExp) {
        // the first tile's counts need its planes, and the second tile's planes must lie in
        // LDS before the first step counts it
        __syncthreads();
        if (cs0 < cs1) {
#pragma unroll
            for (int j = 0; j < NSL; j++) {
                Words w;
                load_words(w, 0, j);
                slice(0, j, w, 0);
                slice(0, j, w, 1);
            }
            stage_planes(1);
            load_planes(min(cs0 + 2 * T, clast));
        }
    }
    __syncthreads();
    // step: tile c0 is computed from `cur`; tile c0 + T is staged into `nxt` and counted (its
    // planes lie in nxt since the step before); the planes of c0 + 2T replace those in `cur`
    // (counted a step ago)
    auto step = [&](int cur, int nxt, int c0) {
        const int c1 = min(c0 + T, clast), c2n = min(c0 + 2 * T, clast), c3 = min(c0 + 3 * T, clast);
        Words w[2];
        load_words(w[0], nxt, 0);
        if (kFine && __builtin_expect(varied, 0)) {
            // the running sums in the tile's units
            const int ty = __builtin_amdgcn_readfirstlane(tile_y(c0));
            const int tg = kG ? __builtin_amdgcn_readfirstlane(tile_g(c0)) : 0;
            if (__builtin_expect(ty != cy || tg != cg, 0)) {
                const int dy = cy - ty, dg = cg - tg;
#pragma unroll
                for (int db = 0; db < 2; db++)
#pragma unroll
                    for (int i = 0; i < 16; i++) {
                        if constexpr (kP) outp[db][i] = ldexpf(outp[db][i], kG ? dg : dy);
                        if constexpr (kG) outg[db][i] = ldexpf(outg[db][i], dy + dg);
                    }
                cy = ty;
                cg = tg;
            }
            stage_scales(c1);
        }
        compute(cur, [&](int i, int half) {
            if (half == 0) {
                if (i + 1 < NSL) load_words(w[(i + 1) & 1], nxt, i + 1);
                __builtin_amdgcn_sched_barrier(0);
                slice(nxt, i, w[i & 1], 0);
            } else {
                slice(nxt, i, w[i & 1], 1);
                // the tile's tensors are staged in turn, each after its loads have had a third
                // or half of a tile's time
                constexpr int gap = 8 * NB / kParts;
                if (i % gap == 0 && i / gap < kParts) {
                    const int part = i / gap;
                    stage(nxt, c1, part);
                    load_part(part + 1 < kParts ? c1 : c2n, part + 1 < kParts ? part + 1 : 0);
                }
                if (i == 2) {
                    stage_planes(cur);
                    load_planes(c3);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        __syncthreads();
    };
    // (two steps per turn: the buffers' addresses are constants)
    bool again = false;
    for (int c0 = cs0; c0 < cs1; c0 += 2 * T) {
        step(0, 1, c0);
        if (c0 + T < cs1) step(1, 0, c0 + T);
        if (kFlush && __builtin_expect(((c0 + 2 * T - cs0) & (kFlushRows<NW> - 1)) == 0 && c0 + 2 * T < cs1, 0)) {
            finish(again);
            again = true;
#pragma unroll
            for (int db = 0; db < 2; db++)
#pragma unroll
                for (int i = 0; i < 16; i++) outp[db][i] = outg[db][i] = 0.f;
        }
    }
    finish(again);
}

__global__ void zero_rows_kernel(uint32_t *__restrict__ p, int64_t words) {
    for (int64_t e = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; e < words;
         e += static_cast<int64_t>(gridDim.x) * blockDim.x)
        p[e] = 0u;
}

// zero `bytes` (a multiple of 4) of an output that no pair reaches
hipError_t zero_rows_async(void *p, int64_t bytes, hipStream_t stream) {
    const int64_t words = bytes / 4;
    if (words == 0) return hipSuccess;
    const int64_t blocks = (words + 255) / 256;
    hipLaunchKernelGGL(zero_rows_kernel, dim3(static_cast<unsigned>(blocks < 4096 ? blocks : 4096)), dim3(256), 0,
                       stream, static_cast<uint32_t *>(p), words);
    return hipGetLastError();
}

// dQ, dK, dV = sums over the splits of their fp32 partial outputs, in split order
template <bool BF16>
__global__ __launch_bounds__(256) void split_sum_kernel(SplitSum a) {
    const int64_t total = a.count4[0] + a.count4[1] + a.count4[2];
    for (int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; t < total;
         t += static_cast<int64_t>(gridDim.x) * 256) {
        const int o = t < a.count4[0] ? 0 : (t < a.count4[0] + a.count4[1] ? 1 : 2);
        const int64_t i = t - (o > 0 ? a.count4[0] : 0) - (o > 1 ? a.count4[1] : 0);
        const int64_t n4 = o == 0 ? a.count4[0] : (o == 1 ? a.count4[1] : a.count4[2]);
        const floatx4 *part = reinterpret_cast<const floatx4 *>(o == 0 ? a.part[0] : (o == 1 ? a.part[1] : a.part[2]));
        void *out = o == 0 ? a.out[0] : (o == 1 ? a.out[1] : a.out[2]);
        floatx4 acc = part[i];
        const int split = o == 0 ? a.split[0] : (o == 1 ? a.split[1] : a.split[2]);
        for (int sp = 1; sp < split; sp++) acc += part[sp * n4 + i];
        if constexpr (BF16) {
            uint2 w;
            w.x = static_cast<uint32_t>(f32_to_bf16(acc[0])) | (static_cast<uint32_t>(f32_to_bf16(acc[1])) << 16);
            w.y = static_cast<uint32_t>(f32_to_bf16(acc[2])) | (static_cast<uint32_t>(f32_to_bf16(acc[3])) << 16);
            reinterpret_cast<uint2 *>(out)[i] = w;
        } else {
            reinterpret_cast<floatx4 *>(out)[i] = acc;
        }
    }
}

int64_t side_blocks(const TileArgs &a, int rows) {
    int64_t n = (a.side[0].n_f + rows - 1) / rows;
    if (a.sides > 1) n += (a.side[1].n_f + rows - 1) / rows;
    return a.bh * n;
}

// Workgroups of a launch: 8 waves (256 fixed rows, one per CU) or 4 (128 rows, two per CU),
// the latter with the streamed rows shared among `split` workgroups where the blocks alone
// would leave CUs idle.  Each is priced by its rounds over 256 CUs (a last round of at most
// one 4-wave workgroup per CU at 0.62 of a full one); 4 waves stage each streamed row
// twice as often, priced at 6%.  (64 heads of 1500 x 1030, bf16: 410 us with 8 waves, 362
// with 4; 32 x 4096 fp32: 1123 and 1190.)
struct TileShape {
    bool wide;  // 8 waves
    int split;
    double rounds;  // rounds of a full CU's work, each over n_s / split streamed rows
};
constexpr int kTileMaxSplit = 16;
constexpr int kTileMinShare = 64;  // streamed rows per share at least

TileShape tile_shape(int64_t blocks8, int64_t blocks4, int64_t n_s, int max_split) {
    if (blocks4 >= 512) {
        const int64_t rem = blocks4 % 512;
        const double t8 = static_cast<double>((blocks8 + 255) / 256);
        const double t4 = 1.06 * (static_cast<double>(blocks4 / 512) + (rem == 0 ? 0.0 : rem <= 256 ? 0.62 : 1.0));
        return {t8 <= t4, 1, t8 <= t4 ? t8 : t4};
    }
    int split = 1;
    while (split < max_split && blocks4 * split * 2 <= 512 && n_s >= static_cast<int64_t>(kTileMinShare) * split * 2)
        split *= 2;
    return {false, split, blocks4 * split <= 256 ? 0.66 : 1.06};
}

template <int WT, int SUM, bool BF16, int NW, int WAVES>
hipError_t launch_tiles_w(const TileArgs &a, hipStream_t stream, const char *name) {
    const int64_t blocks = side_blocks(a, 32 * WAVES) * a.split;
    if (blocks == 0) return hipSuccess;
    // a word per tile of each streamed tensor (YOSO-E: at most 16 KiB; counts: of kFineRows rows)
    const int words = WT == kWeightStar ? 0
                      : WT == kWeightExpect ? (SUM == kSumP ? 1 : 2) * ((a.side[0].n_s + 8 * WAVES - 1) / (8 * WAVES))
                                            : (SUM == kSumP ? 1 : 2) * kFineTiles;
    KernelTimer timer(name, stream);
    hipLaunchKernelGGL((tile_kernel<WT, SUM, BF16, NW, WAVES>), dim3(static_cast<unsigned>(blocks)), dim3(64 * WAVES),
                       (tile_lds<WT, SUM, NW, WAVES>() + 4 * words), stream, a);
    return hipGetLastError();
}

template <int WT, int SUM, bool BF16, int NW>
hipError_t launch_tiles(const TileArgs &a, bool wide, hipStream_t stream, const char *name) {
    // (more than 8 plane words leave too few registers for the 8-wave forms that also take dV
    // or *YOSO's weight)
    if constexpr (NW == 8 || (WT == kWeightCount && SUM == kSumG)) {
        if (wide) return launch_tiles_w<WT, SUM, BF16, NW, 8>(a, stream, name);
    }
    return launch_tiles_w<WT, SUM, BF16, NW, 4>(a, stream, name);
}

// a launch without scratch: no split
template <int WT, int SUM, bool BF16, int NW>
hipError_t launch_tiles_alone(TileArgs &a, hipStream_t stream, const char *name) {
    a.split = 1;
    return launch_tiles<WT, SUM, BF16, NW>(a, tile_shape(side_blocks(a, 256), side_blocks(a, 128), 0, 1).wide, stream,
                                           name);
}

}  // namespace

hipError_t launch_split_sum(const SplitSum &a, bool bf16, hipStream_t stream) {
    const int64_t total = a.count4[0] + a.count4[1] + a.count4[2];
    if (total == 0) return hipSuccess;
    const int64_t blocks = (total + 255) / 256 < 4096 ? (total + 255) / 256 : 4096;
    KernelTimer timer("dense_sum_kernel", stream);
    if (bf16)
        hipLaunchKernelGGL(split_sum_kernel<true>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, a);
    else
        hipLaunchKernelGGL(split_sum_kernel<false>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, stream, a);
    return hipGetLastError();
}

namespace {

// The shapes of the backward's launches (dK and dV; dQ; *YOSO: both in one) and their
// partial outputs in the scratch of t.part_bytes.
struct TilePlan {
    TileShape kv, q;
    bool merged;  // both sides in one launch of the form that also takes dV
    size_t part_bytes;
    bool maxima;  // taken by the prep kernel, not by a scan of each workgroup
};

TilePlan tile_plan(int64_t bh, int64_t n_q, int64_t n_k, bool star, size_t room) {
    auto blocks = [&](int64_t n, int rows) { return bh * ((n + rows - 1) / rows); };
    TilePlan p{};
    // A few heads (both sides together below 512 workgroups of 128 rows) take one launch for
    // both sides, dQ's in the same form: its unused P sum is cheaper than a second launch with
    // most CUs idle (backward, m = 32, tau = 8: 2 x 512 28.9 us in two launches, 20.6 in one; 1 x
    // 2048 43.4 / 34.6, bf16 41.4 / 28.5; 2 x 4096 100 / 91).  Both sides have one split, bounded
    // by the shorter: sides of unlike lengths keep two launches.
    p.merged = !star && blocks(n_q, 128) + blocks(n_k, 128) < 512 && n_q <= 4 * n_k && n_k <= 4 * n_q;
    for (int most = kTileMaxSplit;; most /= 2) {
        if (star || p.merged) {
            p.kv = tile_shape(blocks(n_q, 256) + blocks(n_k, 256), blocks(n_q, 128) + blocks(n_k, 128),
                              n_q < n_k ? n_q : n_k, most);
            p.q = p.kv;
        } else {
            p.kv = tile_shape(blocks(n_k, 256), blocks(n_k, 128), n_q, most);
            p.q = tile_shape(blocks(n_q, 256), blocks(n_q, 128), n_k, most);
        }
        p.part_bytes = 0;
        if (p.q.split > 1) p.part_bytes += static_cast<size_t>(p.q.split) * bh * n_q * D * 4;
        if (p.kv.split > 1) p.part_bytes += static_cast<size_t>(p.kv.split) * bh * n_k * D * 4 * (star ? 1 : 2);
        if (most == 1 || p.part_bytes <= room) break;
    }
    // a scan costs each workgroup one more read of the streamed rows: less than the maxima's
    // own pass while the workgroups are few rounds of short sequences
    p.maxima = p.kv.split > 1 || p.q.split > 1 || n_q >= 2048 || n_k >= 2048;
    return p;
}

}  // namespace

// Fitted to 1 to 64 heads of 300 to 20000 rows, m 1 to 48, tau 4 to 12 (380 shapes; half within 5 to
// 6%, nine in ten within 12%): per streamed row that a CU visits (dK and dV 0.54 of the time, dQ
// 0.46) by plane words, per row of both sides (planes, maxima, outputs), per byte of partial outputs.
double tile_cost(bool bf16, int64_t bh, int64_t n_q, int64_t n_k, int m, int tau, size_t room) {
    const TilePlan p = tile_plan(bh, n_q, n_k, false, room);
    const double rows = p.merged ? 0.54 * p.kv.rounds * static_cast<double>(n_q > n_k ? n_q : n_k) / p.kv.split
                                 : 0.54 * p.kv.rounds * static_cast<double>(n_q) / p.kv.split +
                                       0.46 * p.q.rounds * static_cast<double>(n_k) / p.q.split;
    const int nw = tile_plane_words(m, tau);
    const double row = bf16 ? (nw == 8 ? 0.0862 : nw == 12 ? 0.0987 : 0.120) : (nw == 8 ? 0.116 : nw == 12 ? 0.129 : 0.217);
    return 14.0 + row * rows + (bf16 ? 2.0e-4 : 3.1e-4) * static_cast<double>(bh * (n_q + n_k)) +
           (bf16 ? 6.0e-7 : 7.1e-7) * static_cast<double>(p.part_bytes);
}

// Fitted like tile_cost to 1 to 64 heads of 5 to 32000 rows (300 shapes; half within 6%, nine in ten
// within 20%): the longest workgroups, which stream the longer side, and the work of all.
double tile_star_cost(bool bf16, int64_t bh, int64_t n_q, int64_t n_k, int m, int tau, size_t room) {
    const TilePlan p = tile_plan(bh, n_q, n_k, true, room);
    const double longest = static_cast<double>(n_q > n_k ? n_q : n_k) / p.kv.split;
    const double work = static_cast<double>(bh * ((n_q + 127) / 128 * n_k + (n_k + 127) / 128 * n_q)) / 512.0;
    const int nw = tile_plane_words(m, tau);
    const double words = nw == 8 ? 1.0 : bf16 ? (nw == 12 ? 1.29 : 1.5) : (nw == 12 ? 1.56 : 1.82);
    const double a = (bf16 ? 0.0553 : 0.0711) * longest, b = (bf16 ? 0.103 : 0.113) * work;
    return 20.0 + words * sqrt(a * a + b * b) + 3.0e-4 * static_cast<double>(bh * (n_q + n_k)) +
           (bf16 ? 7.0e-7 : 8.9e-7) * static_cast<double>(p.part_bytes);
}

namespace {

template <bool BF16, int NW>
hipError_t launch_tile_backward(const TileBackward &t, hipStream_t stream) {
    const TilePlan plan = tile_plan(t.bh, t.n_q, t.n_k, t.star, t.part_bytes);
    const int64_t rows_q = t.bh * t.n_q, rows_k = t.bh * t.n_k;
    // Row ranges of a tensor's maxima.  Up to kFineRows rows: only those there are, of 128 rows where
    // the heads alone fill the card (174 x 255 x 112, bf16: 18.6 us with eight ranges, most of them
    // empty, 11.3 with two), else an eighth of the longer side in whole tiles
    // (1 x 512: 4.8 us, with ranges of 128 5.4).
    const int64_t longer = t.n_q > t.n_k ? t.n_q : t.n_k;
    const int fine_per = longer > kFineRows || t.bh > 32
                             ? kFineRows / kMaxParts
                             : static_cast<int>((longer + kMaxParts * kTileRows - 1) / (kMaxParts * kTileRows)) * kTileRows;
    const int parts = longer > kFineRows ? kMaxParts : static_cast<int>((longer + fine_per - 1) / fine_per);
    {
        const int64_t plane_blocks = ((rows_q + rows_k) * (NW == 16 ? 2 : 1) + 255) / 256;
        const int64_t max_blocks = plan.maxima ? t.bh * 4 * parts : 0;
        KernelTimer timer("tile_prep_kernel", stream);
        hipLaunchKernelGGL((tile_prep_kernel<NW, BF16>), dim3(static_cast<unsigned>(plane_blocks + max_blocks)),
                           dim3(256), 0, stream, t.qcodes, t.kcodes, t.qpl, t.kpl, rows_q, rows_k, t.m, t.tau,
                           plane_blocks, t.q, t.dy, t.k, t.v, t.n_q, t.n_k, t.pmax, parts, fine_per);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const int64_t nq = rows_q * D, nk = rows_k * D;
    auto pmax = [&](int i) { return plan.maxima ? t.pmax + i * kMaxParts * D : nullptr; };
    auto tmax = [&](int i) { return t.pmax + t.bh * 4 * kMaxParts * D + i * kFineTiles; };
    TileArgs a{};
    a.bh = t.bh; a.m = t.m; a.tau = t.tau; a.parts = parts;
    TileSide kv{}, q{};
    // keys fixed (a = V), queries streamed (g = dY, y = Q)
    kv.fa = t.v; kv.sg = t.dy; kv.sy = t.q; kv.fpl = t.kpl; kv.spl = t.qpl;
    kv.out_p = t.dv; kv.out_g = t.dk;
    kv.max_g = pmax(1); kv.max_y = pmax(0); kv.tmax_g = tmax(1); kv.tmax_y = tmax(0);
    kv.n_f = static_cast<int>(t.n_k); kv.n_s = static_cast<int>(t.n_q);
    // queries fixed (a = dY), keys streamed (g = V, y = K)
    q.fa = t.dy; q.sg = t.v; q.sy = t.k; q.fpl = t.qpl; q.spl = t.kpl;
    q.out_g = t.dq;
    q.max_g = pmax(3); q.max_y = pmax(2); q.tmax_g = tmax(3); q.tmax_y = tmax(2);
    q.n_f = static_cast<int>(t.n_q); q.n_s = static_cast<int>(t.n_k);
    q.part_g = t.part;
    kv.part_g = t.part + (plan.q.split > 1 ? plan.q.split * nq : 0);
    kv.part_p = kv.part_g + plan.kv.split * nk;
    if (t.star) {
        // *YOSO: both sides the same kernel; x = q . k of the rows as given, streamed as sy
        kv.fx = t.k; kv.out_p = nullptr;
        q.fx = t.q;
        a.side[0] = q; a.side[1] = kv; a.sides = 2; a.split = plan.kv.split;
        e = launch_tiles<kWeightStar, kSumG, BF16, NW>(a, plan.kv.wide, stream, "tile_star_kernel");
    } else if (plan.merged) {
        a.side[0] = kv; a.side[1] = q; a.sides = 2; a.split = plan.kv.split;
        e = launch_tiles<kWeightCount, kSumPG, BF16, NW>(a, plan.kv.wide, stream, "tile_kernel");
    } else {
        a.sides = 1;
        a.side[0] = kv; a.split = plan.kv.split;
        e = launch_tiles<kWeightCount, kSumPG, BF16, NW>(a, plan.kv.wide, stream, "tile_kernel");
        if (e != hipSuccess) return e;
        a.side[0] = q; a.split = plan.q.split;
        e = launch_tiles<kWeightCount, kSumG, BF16, NW>(a, plan.q.wide, stream, "tile_kernel");
    }
    if (e != hipSuccess) return e;
    SplitSum s{};
    s.part[0] = q.part_g; s.out[0] = t.dq; s.split[0] = plan.q.split; s.count4[0] = plan.q.split > 1 ? nq / 4 : 0;
    s.part[1] = kv.part_g; s.out[1] = t.dk; s.split[1] = plan.kv.split; s.count4[1] = plan.kv.split > 1 ? nk / 4 : 0;
    s.part[2] = kv.part_p; s.out[2] = t.dv; s.split[2] = plan.kv.split; s.count4[2] = t.star ? 0 : s.count4[1];
    return launch_split_sum(s, BF16, stream);
}

}  // namespace

int tile_plane_words(int m, int tau) { return m > 32 ? (tau > 8 ? 0 : 16) : (tau > 8 ? 12 : 8); }

hipError_t launch_tile_backward(const TileBackward &t, bool bf16, hipStream_t stream) {
    switch (tile_plane_words(t.m, t.tau)) {
        case 8: return bf16 ? launch_tile_backward<true, 8>(t, stream) : launch_tile_backward<false, 8>(t, stream);
        case 12: return bf16 ? launch_tile_backward<true, 12>(t, stream) : launch_tile_backward<false, 12>(t, stream);
        case 16: return bf16 ? launch_tile_backward<true, 16>(t, stream) : launch_tile_backward<false, 16>(t, stream);
        default: return hipErrorInvalidValue;
    }
}

bool tile_forward_codes(const uint16_t *qcodes, const uint16_t *kcodes, int m, int tau) {
    return tile_plane_words(m, tau) != 0 && m % 8 == 0 &&
           ((reinterpret_cast<uintptr_t>(qcodes) | reinterpret_cast<uintptr_t>(kcodes)) & 15) == 0;
}

hipError_t launch_tile_forward(const uint16_t *qcodes, const uint16_t *kcodes, const void *v, void *y, bool bf16,
                               int64_t bh, int64_t n_q, int64_t n_k, int m, int tau, hipStream_t stream) {
    TileArgs a{};
    TileSide &s = a.side[0];
    s.sy = v; s.fcodes = qcodes; s.scodes = kcodes; s.out_p = y;
    s.n_f = static_cast<int>(n_q); s.n_s = static_cast<int>(n_k);
    a.bh = bh; a.sides = 1; a.m = m; a.tau = tau;
    auto go = [&](auto nw) {
        constexpr int NW = decltype(nw)::value;
        KernelTimer timer("tile_fwd_kernel", stream);  // (beside the name that both dense forms share)
        return bf16 ? launch_tiles_alone<kWeightCount, kSumP, true, NW>(a, stream, "dense_fwd_kernel")
                    : launch_tiles_alone<kWeightCount, kSumP, false, NW>(a, stream, "dense_fwd_kernel");
    };
    switch (tile_plane_words(m, tau)) {
        case 8: return go(std::integral_constant<int, 8>{});
        case 12: return go(std::integral_constant<int, 12>{});
        case 16: return go(std::integral_constant<int, 16>{});
        default: return hipErrorInvalidValue;
    }
}

namespace {

// The scale of YOSO-E's P before its split: the power of a factor pbase of the base.  P is at
// most 1 and the pair ends at 2^-24, so pbase^tau lies just below fp16's largest number, for
// every tau: a row whose cosines are all negative has only small P (2^15 a power of
// two per factor leaves as little as 2^8 at tau = 8: Y of rows at cosines about -0.8 is then 1.6e-5
// off instead of 1.7e-6).  pbase is a multiple of 1/32, so that half of it is exact, and pinv
// divides by the power as the kernel rounds it, so that P = 1 comes out as 1.
void expect_scale(TileArgs &a) {
    auto power = [&](float x) {  // ipow's order of products
        float r = x;
        int bit = 16;
        while (bit > a.tau) bit >>= 1;
        for (bit >>= 1; bit > 0; bit >>= 1) r = (a.tau & bit) ? (r * r) * x : r * r;
        return r;
    };
    int k = 32;
    for (int step = 1 << 20; step > 0; step >>= 1)
        if (power((k + step) / 32.0f) <= 65000.0f) k += step;
    a.pbase = static_cast<float>(k) / 32.0f;
    a.pinv = 1.0f / power(a.pbase);
}

}  // namespace

hipError_t launch_expect_forward(const void *q, const void *k, const void *v, void *y, bool bf16, int64_t bh,
                                 int64_t n_q, int64_t n_k, int tau, hipStream_t stream) {
    if (bh == 0 || n_q == 0) return hipSuccess;
    if (n_k == 0) return zero_rows_async(y, bh * n_q * D * (bf16 ? 2 : 4), stream);
    if (expect_blocks_apply(kExpectForward, bf16, bh, n_q, n_k)) {
        ExpectBlocks e{};
        e.xr = q; e.xc = k; e.yc = v; e.out1 = y;
        e.bh = bh; e.n_r = static_cast<int>(n_q); e.n_c = static_cast<int>(n_k); e.tau = tau;
        return launch_expect_blocks(kExpectForward, e, bf16, stream);
    }
    TileArgs a{};
    a.side[0].fx = q; a.side[0].sx = k; a.side[0].sy = v; a.side[0].out_p = y;
    a.side[0].n_f = static_cast<int>(n_q); a.side[0].n_s = static_cast<int>(n_k);
    a.bh = bh; a.sides = 1; a.tau = tau; a.m = 1; a.split = 1;
    expect_scale(a);
    return bf16 ? launch_tiles_alone<kWeightExpect, kSumP, true, 8>(a, stream, "expect_fwd_kernel")
                : launch_tiles_alone<kWeightExpect, kSumP, false, 8>(a, stream, "expect_fwd_kernel");
}

hipError_t launch_expect_backward(const void *q, const void *k, const void *v, const void *dy, void *dq, void *dk,
                                  void *dv, bool bf16, int64_t bh, int64_t n_q, int64_t n_k, int tau,
                                  hipStream_t stream) {
    if (bh == 0) return hipSuccess;
    const int64_t e = bf16 ? 2 : 4;
    hipError_t err;
    if (n_q == 0 || n_k == 0) {
        if ((err = zero_rows_async(dq, bh * n_q * D * e, stream)) != hipSuccess) return err;
        if ((err = zero_rows_async(dk, bh * n_k * D * e, stream)) != hipSuccess) return err;
        return zero_rows_async(dv, bh * n_k * D * e, stream);
    }
    ExpectBlocks x{};
    x.bh = bh; x.tau = tau;
    // keys fixed, queries streamed: dV and dK
    TileArgs a{};
    a.bh = bh; a.sides = 1; a.tau = tau; a.m = 1; a.split = 1;
    expect_scale(a);
    TileSide &s = a.side[0];
    s.fx = k; s.fa = v; s.sx = q; s.sg = dy; s.sy = q; s.out_p = dv; s.out_g = dk;
    s.n_f = static_cast<int>(n_k); s.n_s = static_cast<int>(n_q);
    if (expect_blocks_apply(kExpectKV, bf16, bh, n_k, n_q)) {
        x.xr = k; x.ar = v; x.xc = q; x.bc = dy; x.yc = q; x.out1 = dv; x.out2 = dk;
        x.n_r = static_cast<int>(n_k); x.n_c = static_cast<int>(n_q);
        err = launch_expect_blocks(kExpectKV, x, bf16, stream);
    } else {
        err = bf16 ? launch_tiles_alone<kWeightExpect, kSumPG, true, 8>(a, stream, "expect_bwd_kv_kernel")
                   : launch_tiles_alone<kWeightExpect, kSumPG, false, 8>(a, stream, "expect_bwd_kv_kernel");
    }
    if (err != hipSuccess) return err;
    // queries fixed, keys streamed: dQ
    if (expect_blocks_apply(kExpectQ, bf16, bh, n_q, n_k)) {
        x.xr = q; x.ar = dy; x.xc = k; x.bc = v; x.yc = k; x.out1 = nullptr; x.out2 = dq;
        x.n_r = static_cast<int>(n_q); x.n_c = static_cast<int>(n_k);
        return launch_expect_blocks(kExpectQ, x, bf16, stream);
    }
    s = TileSide{};
    s.fx = q; s.fa = dy; s.sx = k; s.sg = v; s.sy = k; s.out_g = dq;
    s.n_f = static_cast<int>(n_q); s.n_s = static_cast<int>(n_k);
    return bf16 ? launch_tiles_alone<kWeightExpect, kSumG, true, 8>(a, stream, "expect_bwd_q_kernel")
                : launch_tiles_alone<kWeightExpect, kSumG, false, 8>(a, stream, "expect_bwd_q_kernel");
}

}  // namespace yoso

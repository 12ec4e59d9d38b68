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
// What bounds it: per pair about 13 (C) to 25 (P, N) vector instructions and 12 to 32
// MFMAs per 1024 pairs, nearly in balance on a SIMD.  Two waves share a SIMD; half of the
// waves prepare the next tile (convert and stage its rows, count its pairs) before their
// MFMA work on the present one and half after it, so that the two do not compete for the
// same unit.  Tiles and counts are double buffered in LDS: one barrier per tile.
//
// Precision: fp32 operands as fp16 (hi, lo) pairs and three products, as everywhere in
// this library; bf16 operands, scaled by powers of two, are exact as hi alone (cosine rows,
// which are normalised, keep both).  Scales, all powers of two but the first:
//   cosine rows     unit length times 2^4
//   fixed rows a    each row by 2^(6 - e), ||a|| < 2^e
//   streamed rows   each head's tensor by 2^(13 - e), max |x| < 2^e (found by a first scan)
//   weights         |G| < 2^22, times C (or N, P) and a constant that keeps W below 2^15
#include "common.h"
#include "launch.h"
#include "timing.h"

namespace yoso {

namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef _Float16 half2v __attribute__((ext_vector_type(2)));

enum : int { kWeightCount = 0, kWeightStar = 1, kWeightExpect = 2 };
// which sums: the P (or C) weighted one, the G weighted one, or both
enum : int { kSumP = 0, kSumPG = 1, kSumG = 2 };

constexpr float kCosScale = 16.0f;   // cosine rows: unit length times 2^4
constexpr int kFixedExp = 6;         // fixed rows: norm below 2^6
constexpr float kNearFloor = 1.0f / 64.0f;  // *YOSO: 1 - x^2 is raised to at least 1/64

struct TileSide {
    const void *fx, *fa;         // fixed side: cosine (or x) rows, rows of G
    const void *sx, *sg, *sy;    // streamed side: cosine rows, rows of G, rows summed
    const uint32_t *fpl, *spl;   // bit planes of the codes [bh][n][NW] (C, N)
    void *out_p, *out_g;         // P- (C-) weighted sum of sg (forward: of sy); G-weighted sum of sy
    float *part_p, *part_g;      // split > 1: their fp32 partial sums [split][bh][n_f][64]
    int n_f, n_s;
};

struct TileArgs {
    TileSide side[2];
    int64_t bh;
    int sides, m, tau;
    int split;  // workgroups per block of fixed rows, each streaming a contiguous share
};

// A constant the compiler does not see through: a multiply-add by it stays one, so that
// it can take an fp16 operand in place (v_fma_mix_f32) instead of converting it first.
__device__ __forceinline__ float opaque(float x) {
    asm("" : "+s"(x));
    return x;
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

// Streamed tiles: rows of 256 bytes [hi 64 | lo 64], 16-byte chunk c of row r at slot
// c ^ f(r).  f is a bijection of r mod 16, so that 16 rows read at one chunk hit distinct
// banks, and f >> 2 differs within every 4 aligned rows, so that a transposing read (4
// rows x 4 chunks per half-wave) does too.
__device__ __forceinline__ uint32_t tswz(int row) {
    return static_cast<uint32_t>(((row & 3) << 2) | ((row >> 2) & 3));
}

__device__ __forceinline__ half4 tile_tr(const unsigned char *p) {
    typedef short short4v __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) short4v lds_short4;
    return __builtin_bit_cast(half4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4 *)(p)));
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
template <int WT, int SUM, int WAVES>
constexpr int tile_lds() {
    constexpr int T = 8 * WAVES;
    constexpr int tiles = 1 + (SUM != kSumP ? 1 : 0) + (WT == kWeightExpect ? 1 : 0);
    constexpr int counts = WT == kWeightExpect ? 0 : 32 * WAVES * T * 2;
    return 2 * (tiles * T * 256 + counts);
}

// NW: plane words per row (8: tau <= 8; 12: tau <= 12; 16: two words per plane, tau <= 8)
template <int WT, int SUM, bool BF16, int NW, int WAVES>
__global__ __launch_bounds__(64 * WAVES) __attribute__((amdgpu_waves_per_eu(2, 2))) void tile_kernel(TileArgs args) {
    constexpr bool kP = SUM != kSumG, kG = SUM != kSumP;
    constexpr bool kExp = WT == kWeightExpect, kStar = WT == kWeightStar;
    constexpr bool kX = WT != kWeightCount;  // a scalar product x beside G
    constexpr int T = 8 * WAVES;             // streamed rows per tile
    constexpr int NB = T / 32;               // 32-row blocks per tile
    constexpr int TB = T * 256;              // LDS bytes of one tensor's tile
    constexpr int kTiles = 1 + (kG ? 1 : 0) + (kExp ? 1 : 0);
    constexpr int CROW = T * 2;              // LDS bytes of a fixed row's counts
    constexpr int CB = kExp ? 0 : 32 * WAVES * CROW;
    constexpr int BUF = kTiles * TB + CB;
    // tile order within a buffer: summed rows, rows of G, cosine rows, counts
    constexpr int OY = 0, OG = TB, OX = kStar ? OY : (kG ? 2 : 1) * TB, OC = kTiles * TB;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ float wmax[2][WAVES];

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
    Raw<BF16> ry, rg, rx;
    auto load_tile = [&](int c0) {
        const int64_t off = sbase + static_cast<int64_t>(min(c0 + srow, ns - 1)) * D;
        raw_load<BF16>(ry, a.sy, off);
        if constexpr (kG) raw_load<BF16>(rg, a.sg, off);
        if constexpr (kExp) raw_load<BF16>(rx, a.sx, off);
    };

    // ---- the streamed tensors' largest |value| over the head (every split scans all of
    // it, so that the scales, and the results, do not depend on the share)
    float mg = 0.f, my = 0.f;
    for (int c = srow; c < ns; c += 4 * T) {
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
            for (int e = 0; e < 8; e++) my = fmaxf(my, fabsf(v[e]));
            if constexpr (kG) {
                raw_values<BF16>(w[i], v);
#pragma unroll
                for (int e = 0; e < 8; e++) mg = fmaxf(mg, fabsf(v[e]));
            }
        }
    }
    load_tile(cs0);
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
    if constexpr (kG) {
        float v[4][8], ss = 0.f;
#pragma unroll
        for (int s = 0; s < 4; s++) {
            load8<BF16>(a.fa, foff + 16 * s, v[s]);
#pragma unroll
            for (int i = 0; i < 8; i++) ss = fmaf(v[s][i], v[s][i], ss);
        }
        ss += __shfl_xor(ss, 32);
        int e2 = 0;
        if (ss > 0.f) frexpf(ss, &e2);  // ss < 2^e2: the norm is below 2^ceil(e2/2)
        ea = min(max((e2 + 1) >> 1, -60), 60);
#pragma unroll
        for (int s = 0; s < 4; s++) split8_pk(v[s], ldexpf(1.0f, kFixedExp - ea), arh[s], arl[s]);
    }
    if constexpr (kX) {
        float v[4][8], ss = 0.f;
#pragma unroll
        for (int s = 0; s < 4; s++) {
            load8<BF16>(a.fx, foff + 16 * s, v[s]);
#pragma unroll
            for (int i = 0; i < 8; i++) ss = fmaf(v[s][i], v[s][i], ss);
        }
        ss += __shfl_xor(ss, 32);
        float sc;
        if constexpr (kExp) {
            sc = ss > 0.f ? kCosScale / sqrtf(ss) : 0.f;
        } else {
            int e2 = 0;
            if (ss > 0.f) frexpf(ss, &e2);
            ex = min(max((e2 + 1) >> 1, -60), 60);
            sc = ldexpf(1.0f, kFixedExp - ex);
        }
#pragma unroll
        for (int s = 0; s < 4; s++) split8_pk(v[s], sc, xrh[s], xrl[s]);
    }

    // ---- counting role: lane = fixed row 64 (wave mod WAVES/2) + lane, partners T/2 (wave /
    // (WAVES/2)) + [0, T/2) of a tile, whose plane words are wave-uniform (scalar loads)
    constexpr int HW = WAVES / 2;
    const int crow = 64 * (wave % HW) + lane, cpart = wave / HW;
    uint32_t qp[kExp ? 1 : NW];
    if constexpr (!kExp) {
        const uint4 *src = reinterpret_cast<const uint4 *>(a.fpl + (b * nf + min(r0 + crow, nf - 1)) * NW);
#pragma unroll
        for (int j = 0; j < NW / 4; j++) {
            const uint4 w4 = src[j];
            qp[4 * j] = w4.x; qp[4 * j + 1] = w4.y; qp[4 * j + 2] = w4.z; qp[4 * j + 3] = w4.w;
        }
    }
    // the largest count: m, or tau m times the largest weight 8/pi < 2.55
    const int cmax = kStar ? args.tau * args.m : args.m;
    int kc = 0;
    while ((1 << kc) < cmax) kc++;  // 2^kc >= cmax
    // C is kept as C 2^-(7 + kc) (an exact fp16 number): |G| < 2^22, so W < 2^15; *YOSO keeps
    // N itself and scales the weight
    const float cscale = ldexpf(1.0f, -(7 + kc));

    __syncthreads();
    float hy = 0.f, hg = 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; w++) {
        hy = fmaxf(hy, wmax[0][w]);
        hg = fmaxf(hg, wmax[1][w]);
    }
    const int ey = __builtin_amdgcn_readfirstlane(pow2_above(hy));
    const int eg = kG ? __builtin_amdgcn_readfirstlane(pow2_above(hg)) : 0;
    const float scy = ldexpf(1.0f, 13 - ey), scg = ldexpf(1.0f, 13 - eg);

    // convert and stage the tile held in the raw registers (rows past cs1 as zeros)
    auto stage = [&](unsigned char *buf, int c0) {
        const bool ok = c0 + srow < cs1;
        unsigned char *row = buf + srow * 256;
        const uint32_t f = tswz(srow);
        auto put = [&](unsigned char *t, const Raw<BF16> &r, float scale, bool lo_too, bool unit) {
            float v[8];
            raw_values<BF16>(r, v);
#pragma unroll
            for (int i = 0; i < 8; i++) v[i] = ok ? v[i] : 0.f;
            if (unit) {
                float ss = 0.f;
#pragma unroll
                for (int i = 0; i < 8; i++) ss = fmaf(v[i], v[i], ss);
                ss = group_sum(ss, 8);  // the row's 8 threads
                scale = ss > 0.f ? kCosScale / sqrtf(ss) : 0.f;
            }
            half8 h, l;
            split8_pk(v, scale, h, l);
            *reinterpret_cast<half8 *>(t + ((soct ^ f) << 4)) = h;
            if (lo_too) *reinterpret_cast<half8 *>(t + (((8 + soct) ^ f) << 4)) = l;
        };
        put(row + OY, ry, scy, !BF16, false);
        if constexpr (kG) put(row + OG, rg, scg, !BF16, false);
        if constexpr (kExp) put(row + OX, rx, 1.0f, true, true);
    };

    // counts of the tile at c0: the codes' differing hashes are OR_t (plane_t(q) ^ plane_t(k))
    auto count = [&](unsigned char *buf, int c0) {
        unsigned char *crow_lds = buf + OC + crow * CROW;
        const uint32_t f = T == 64 ? (crow & 7) : ((crow >> 2) & 3);
        const uint32_t *pl = a.spl + (b * ns + c0 + (T / 2) * cpart) * NW;
#pragma unroll
        for (int s = 0; s < T / 32; s++) {  // 16 partners at a time
            half2v c2[8];
#pragma unroll
            for (int p = 0; p < 16; p += 2) {
                uint32_t u[2];
#pragma unroll
                for (int i = 0; i < 2; i++) {
                    const uint32_t *w = pl + (16 * s + p + i) * NW;
                    uint32_t d[2] = {0u, 0u}, d2[2] = {0u, 0u};
#pragma unroll
                    for (int j = 0; j < NW; j++) {
                        const int z = NW == 16 ? j & 1 : 0;
                        if constexpr (kStar) {
                            const uint32_t x = qp[j] ^ w[j];
                            d2[z] |= d[z] & x;  // hashes with a second differing bit
                            d[z] |= x;
                        } else {
                            d[z] |= qp[j] ^ w[j];
                        }
                    }
                    if constexpr (kStar) {
                        // tau (m - differing) + (differing in one bit only)
                        const int e = __builtin_popcount(d[0]) + (NW == 16 ? __builtin_popcount(d[1]) : 0);
                        const int one = __builtin_popcount(d[0] & ~d2[0]) +
                                        (NW == 16 ? __builtin_popcount(d[1] & ~d2[1]) : 0);
                        u[i] = 0x6400u + static_cast<uint32_t>(args.tau * (args.m - e) + one);  // fp16 1024 + N
                    } else {
                        u[i] = 0x6400u + static_cast<uint32_t>(__builtin_popcount(d[0]) +
                                                               (NW == 16 ? __builtin_popcount(d[1]) : 0));
                    }
                }
                const half2v c = __builtin_bit_cast(half2v, u[0] | (u[1] << 16));
                // fp16 1024 + k holds k in its low bits; both steps are exact
                if constexpr (kStar) {
                    c2[p / 2] = c - half2v{static_cast<_Float16>(1024.0f), static_cast<_Float16>(1024.0f)};
                } else {
                    const _Float16 top = static_cast<_Float16>(1024.0f + static_cast<float>(args.m));
                    const _Float16 cs = static_cast<_Float16>(cscale);
                    c2[p / 2] = (half2v{top, top} - c) * half2v{cs, cs};
                }
            }
            // element e of half g holds partner 8 (e / 4) + 4 g + e % 4: pairs (2g, 2g+1), (4+2g, 5+2g)
#pragma unroll
            for (int g = 0; g < 2; g++) {
                half8 h;
#pragma unroll
                for (int e = 0; e < 8; e++) {
                    const int p = 8 * (e / 4) + 4 * g + e % 4;
                    h[e] = c2[p / 2][p & 1];
                }
                const uint32_t chunk = 2 * ((T / 32) * cpart + s) + g;
                *reinterpret_cast<half8 *>(crow_lds + ((chunk ^ f) << 4)) = h;
            }
        }
    };

    // ---- block products.  A operand of the scalar products: lane (l31, hh) = streamed row
    // 32 k + l31, dims 16 s + 8 hh + [0, 8)
    const uint32_t fr = tswz(l31);
    auto rows_op = [&](const unsigned char *t, int k, int s, int lo) {
        return *reinterpret_cast<const half8 *>(t + (32 * k + l31) * 256 +
                                                ((static_cast<uint32_t>(8 * lo + 2 * s + hh) ^ fr) << 4));
    };
    // A operand of the sums: lane = dim 32 db + l31; element e of half hh is streamed row
    // 32 k + 16 s + 8 (e / 4) + 4 hh + e % 4, the rows whose weights register 8 s + e of the
    // lane's block result holds.  ds_read_b64_tr_b16 gives destination lane 4a+b of a 16-lane
    // group element b of the 8 bytes addressed by source lanes 4i+a (i = 0..3).
    const int l15 = lane & 15, ti = l15 >> 2, ta = l15 & 3, tg = (lane >> 4) & 1;
    auto sum_op = [&](const unsigned char *t, int k, int s, int db, int lo) {
        const uint32_t ch = static_cast<uint32_t>(8 * lo + 4 * db + 2 * tg + (ta >> 1));
        const int row = 32 * k + 16 * s + 4 * hh + ti;
        const half4 x = tile_tr(t + row * 256 + ((ch ^ tswz(4 * hh + ti)) << 4) + 8 * (ta & 1));
        const half4 y = tile_tr(t + (row + 8) * 256 + ((ch ^ tswz(8 + 4 * hh + ti)) << 4) + 8 * (ta & 1));
        return __builtin_shufflevector(x, y, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    // (the forward has registers to spare: its hi*lo products accumulate apart, so that the
    // large sums are rounded once per 16 rows instead of three times)
    floatx16 outp[2], outg[2], outl[2];
#pragma unroll
    for (int db = 0; db < 2; db++)
#pragma unroll
        for (int i = 0; i < 16; i++) outp[db][i] = outg[db][i] = outl[db][i] = 0.f;

    // YOSO-E: p = (base 2^kt)^tau <= 2^15, base = 1 - arccos(c)/pi.  Two polynomials, both
    // least squares at Chebyshev nodes.  Where every |c| of a block is at most 1/2 (almost
    // all blocks of unclustered rows): 1/2 + arcsin(c)/pi = 1/2 + c A(c^2), A of degree 5,
    // |error| < 7e-9.  Else, with u = 1 - |c|: arccos(|c|)/pi = sqrt(u) Q(u), Q of degree 7,
    // relative error 2e-8.
    const int kt = kExp ? 15 / args.tau : 0;
    const float bs = ldexpf(1.0f, kt);
    constexpr float c2 = kCosScale * kCosScale;  // a block's S is c * c2
    float ca[6] = {0.31830987334251404f, 0.05305203050374985f, 0.023855842649936676f,
                   0.014495517127215862f, 0.007610586937516928f, 0.013545230962336063f};
    float cq[8] = {0.45015814900398254f, 0.037513915449380875f, 0.008425663225352764f, 0.00262420903891325f,
                   0.00044531628373079f, 0.0011004807893186808f, -0.0006614952581003308f, 0.0003937508736271411f};
    {
        float f = bs / c2;
#pragma unroll
        for (int i = 0; i < 6; i++) {
            ca[i] *= f;
            f /= c2 * c2;
        }
#pragma unroll
        for (int i = 0; i < 8; i++) cq[i] *= bs;
    }
    // W = G p wp: |G| < 2^22, p <= 2^(kt tau)
    const float wp = ldexpf(1.0f, -(7 + kt * args.tau));
    // *YOSO: x = S 2^(ex - 6) 2^(ey - 13); weight (s / pi) / sqrt(max(1 - x^2, 1/64)), at most s 2.55
    const float xs = kStar ? ldexpf(1.0f, ex - kFixedExp + ey - 13) : 0.f;
    const float sw = 0.31830988618379067f * ldexpf(1.0f, -(7 + kc + 2));

    const float zero = opaque(0.0f);
    auto split_w = [&](const float w[8], half8 &hi, half8 &lo) { split8_pk(w, 1.0f, hi, lo); };
    auto dot = [&](const unsigned char *t, int k, const half8 fh[4], const half8 fl[4], bool lo) {
        floatx16 acc;
#pragma unroll
        for (int i = 0; i < 16; i++) acc[i] = 0.f;
#pragma unroll
        for (int s = 0; s < 4; s++) {
            const half8 h = rows_op(t, k, s, 0);
            acc = mfma32(h, fh[s], acc);
            if (lo) {
                acc = mfma32(h, fl[s], acc);
                acc = mfma32(rows_op(t, k, s, 1), fh[s], acc);
            }
        }
        return acc;
    };

    auto compute = [&](const unsigned char *buf) {
#pragma unroll
        for (int k = 0; k < NB; k++) {
            floatx16 p;
            if constexpr (kX) p = dot(buf + OX, k, xrh, xrl, kExp || !BF16);
            floatx16 g;
            if constexpr (kG) g = dot(buf + OG, k, arh, arl, !BF16);
            if constexpr (kExp) {
                float most = 0.f;
#pragma unroll
                for (int i = 0; i < 16; i += 2) most = fmaxf(fmaxf(most, fabsf(p[i])), fabsf(p[i + 1]));
                if (__builtin_amdgcn_ballot_w64(most > 0.5f * c2) == 0) {
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
                        const float u = __saturatef(fmaf(-fabsf(p[i]), 1.0f / c2, 1.0f));
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
#pragma unroll
            for (int s = 0; s < 2; s++) {
                half8 c16;
                if constexpr (!kExp) {
                    const int cr = 32 * wave + l31;
                    const uint32_t f = T == 64 ? (cr & 7) : ((cr >> 2) & 3);
                    c16 = *reinterpret_cast<const half8 *>(buf + OC + cr * CROW +
                                                           ((static_cast<uint32_t>(4 * k + 2 * s + hh) ^ f) << 4));
                }
                if constexpr (kP) {
                    // FWD sums y, the key side's backward sums g (dV from dY)
                    const unsigned char *t = buf + (kG ? OG : OY);
                    half8 ph, pl;
                    if constexpr (kExp) {
                        float w[8];
#pragma unroll
                        for (int e = 0; e < 8; e++) w[e] = p[8 * s + e];
                        split_w(w, ph, pl);
                    } else {
                        ph = c16;
                    }
#pragma unroll
                    for (int db = 0; db < 2; db++) {
                        const half8 th = sum_op(t, k, s, db, 0);
                        floatx16 &ol = kG ? outp[db] : outl[db];
                        outp[db] = mfma32(th, ph, outp[db]);
                        if constexpr (kExp) ol = mfma32(th, pl, ol);
                        if constexpr (!BF16) ol = mfma32(sum_op(t, k, s, db, 1), ph, ol);
                    }
                }
                if constexpr (kG) {
                    float w[8];
#pragma unroll
                    for (int e = 0; e < 8; e++) {
                        const int i = 8 * s + e;
                        if constexpr (kExp) {
                            w[e] = g[i] * wp * p[i];
                        } else if constexpr (kStar) {
                            const float x = p[i] * xs;
                            const float z = fmaxf(fmaf(-x, x, 1.0f), kNearFloor);
                            w[e] = g[i] * (static_cast<float>(c16[e]) * (__builtin_amdgcn_rsqf(z) * sw));
                        } else {
                            w[e] = fmaf(g[i], static_cast<float>(c16[e]), zero);
                        }
                    }
                    half8 wh, wl;
                    split_w(w, wh, wl);
#pragma unroll
                    for (int db = 0; db < 2; db++) {
                        const half8 th = sum_op(buf + OY, k, s, db, 0);
                        outg[db] = mfma32(th, wh, outg[db]);
                        outg[db] = mfma32(th, wl, outg[db]);
                        if constexpr (!BF16) outg[db] = mfma32(sum_op(buf + OY, k, s, db, 1), wh, outg[db]);
                    }
                }
            }
        }
    };

    // ---- the pipeline: tile t is computed while t + 1 is staged and counted and t + 2 loaded
    if (cs0 < cs1) {
        stage(smem, cs0);
        if constexpr (!kExp) count(smem, cs0);
        load_tile(cs0 + T);
    }
    __syncthreads();
    const bool early = wave < HW;
    auto step = [&](unsigned char *cur, unsigned char *nxt, int c0) {
        const bool more = c0 + T < cs1;
        auto ahead = [&]() {
            stage(nxt, c0 + T);
            load_tile(c0 + 2 * T);
            if constexpr (!kExp) count(nxt, c0 + T);
        };
        if (early && more) ahead();
        compute(cur);
        if (!early && more) ahead();
        __syncthreads();
    };
    // (two steps per turn: the buffers' addresses are constants)
    for (int c0 = cs0; c0 < cs1; c0 += 2 * T) {
        step(smem, smem + BUF, c0);
        if (c0 + T < cs1) step(smem + BUF, smem, c0 + T);
    }

    // ---- outputs: lane (l31, hh) holds out[row l31][32 db + 8 u + 4 hh + (0..3)] in registers 4u .. 4u+3
    if (frow >= nf) return;
    auto put = [&](void *dst, float *part, const floatx16 o[2], float sc) {
#pragma unroll
        for (int db = 0; db < 2; db++)
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int64_t off = (b * nf + frow) * D + 32 * db + 8 * u + 4 * hh;
                const float x0 = o[db][4 * u] * sc, x1 = o[db][4 * u + 1] * sc, x2 = o[db][4 * u + 2] * sc,
                            x3 = o[db][4 * u + 3] * sc;
                if (split > 1) {
                    *reinterpret_cast<float4 *>(part + sp * (args.bh * nf * D) + off) = make_float4(x0, x1, x2, x3);
                } else if constexpr (BF16) {
                    uint2 w;
                    w.x = static_cast<uint32_t>(f32_to_bf16(x0)) | (static_cast<uint32_t>(f32_to_bf16(x1)) << 16);
                    w.y = static_cast<uint32_t>(f32_to_bf16(x2)) | (static_cast<uint32_t>(f32_to_bf16(x3)) << 16);
                    *reinterpret_cast<uint2 *>(static_cast<uint16_t *>(dst) + off) = w;
                } else {
                    *reinterpret_cast<float4 *>(static_cast<float *>(dst) + off) = make_float4(x0, x1, x2, x3);
                }
            }
    };
    if constexpr (kP) {
        const int e1 = kG ? eg : ey;
        const float sc = kExp ? ldexpf(1.0f, e1 - 13 - kt * args.tau)
                              : ldexpf(1.0f / static_cast<float>(args.m), e1 - 13 + 7 + kc);
        if constexpr (!kG) {
            outp[0] += outl[0];
            outp[1] += outl[1];
        }
        put(a.out_p, a.part_p, outp, sc);
    }
    if constexpr (kG) {
        const int e = (eg - 13) + (ea - kFixedExp) + (ey - 13);
        const float half_tau = 0.5f * static_cast<float>(args.tau);
        const float sc = kExp    ? ldexpf(half_tau, e + 7)
                         : kStar ? ldexpf(1.0f / static_cast<float>(args.m), e + 7 + kc + 2)
                                 : ldexpf(half_tau / static_cast<float>(args.m), e + 7 + kc);
        put(a.out_g, a.part_g, outg, sc);
    }
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

int64_t side_blocks(const TileArgs &a, int rows) {
    int64_t n = (a.side[0].n_f + rows - 1) / rows;
    if (a.sides > 1) n += (a.side[1].n_f + rows - 1) / rows;
    return a.bh * n;
}

template <int WT, int SUM, bool BF16, int NW, int WAVES>
hipError_t launch_tiles_w(const TileArgs &a, hipStream_t stream, const char *name) {
    const int64_t blocks = side_blocks(a, 32 * WAVES) * a.split;
    if (blocks == 0) return hipSuccess;
    KernelTimer timer(name, stream);
    hipLaunchKernelGGL((tile_kernel<WT, SUM, BF16, NW, WAVES>), dim3(static_cast<unsigned>(blocks)), dim3(64 * WAVES),
                       (tile_lds<WT, SUM, WAVES>()), stream, a);
    return hipGetLastError();
}

template <int WT, int SUM, bool BF16, int NW>
hipError_t launch_tiles(const TileArgs &a, hipStream_t stream, const char *name) {
    return side_blocks(a, 256) >= 256 ? launch_tiles_w<WT, SUM, BF16, NW, 8>(a, stream, name)
                                      : launch_tiles_w<WT, SUM, BF16, NW, 4>(a, stream, name);
}

}  // namespace

hipError_t launch_expect_forward(const void *q, const void *k, const void *v, void *y, bool bf16, int64_t bh,
                                 int64_t n_q, int64_t n_k, int tau, hipStream_t stream) {
    if (bh == 0 || n_q == 0) return hipSuccess;
    if (n_k == 0) return zero_rows_async(y, bh * n_q * D * (bf16 ? 2 : 4), stream);
    TileArgs a{};
    a.side[0].fx = q; a.side[0].sx = k; a.side[0].sy = v; a.side[0].out_p = y;
    a.side[0].n_f = static_cast<int>(n_q); a.side[0].n_s = static_cast<int>(n_k);
    a.bh = bh; a.sides = 1; a.tau = tau; a.m = 1; a.split = 1;
    return bf16 ? launch_tiles<kWeightExpect, kSumP, true, 8>(a, stream, "expect_fwd_kernel")
                : launch_tiles<kWeightExpect, kSumP, false, 8>(a, stream, "expect_fwd_kernel");
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
    // keys fixed, queries streamed: dV and dK
    TileArgs a{};
    a.bh = bh; a.sides = 1; a.tau = tau; a.m = 1; a.split = 1;
    TileSide &s = a.side[0];
    s.fx = k; s.fa = v; s.sx = q; s.sg = dy; s.sy = q; s.out_p = dv; s.out_g = dk;
    s.n_f = static_cast<int>(n_k); s.n_s = static_cast<int>(n_q);
    err = bf16 ? launch_tiles<kWeightExpect, kSumPG, true, 8>(a, stream, "expect_bwd_kv_kernel")
               : launch_tiles<kWeightExpect, kSumPG, false, 8>(a, stream, "expect_bwd_kv_kernel");
    if (err != hipSuccess) return err;
    // queries fixed, keys streamed: dQ
    s = TileSide{};
    s.fx = q; s.fa = dy; s.sx = k; s.sg = v; s.sy = k; s.out_g = dq;
    s.n_f = static_cast<int>(n_q); s.n_s = static_cast<int>(n_k);
    return bf16 ? launch_tiles<kWeightExpect, kSumG, true, 8>(a, stream, "expect_bwd_q_kernel")
                : launch_tiles<kWeightExpect, kSumG, false, 8>(a, stream, "expect_bwd_q_kernel");
}

}  // namespace yoso

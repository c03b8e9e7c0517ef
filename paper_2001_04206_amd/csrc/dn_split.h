// fp32 contractions on the f16 matrix cores.
//
// scale x = h + 2^-11 l, h the f16 nearest to scale x and l the f16 nearest to 2^11 times the rest, keeps 22 to 23 of
// an fp32 number's 24 bits.  A product is then h h' + 2^-11 (h l' + l h') (l l' is below the rounding): three f16
// products, each exact, summed in fp32 by v_mfma_f32_32x32x16_f16, h h' in one accumulator and the two small ones in
// another.  Three of those instructions cover sixteen k values in 96 cycles where v_mfma_f32_32x32x2_f32 needs 512,
// and the sum is rounded once per sixteen k instead of eight times.
//
// (Single precision from half precision products, the rest scaled up and summed apart: Ootomo and Yokota, "Recovering
// single precision accuracy from Tensor Cores while surpassing the FP32 theoretical peak performance", 2022.)
//
// f16 has three fewer bits of exponent than fp32, hence the scales: a power of two for every row of either operand, which
// each wave chooses from the numbers it meets (the row's largest so far lies in [2^11, 2^15], and the accumulators
// follow when a number no longer fits).  Nothing overflows.  A scaled number keeps its 22 to 23 bits down to 2^-14, which is
// 2^-25 of the row's largest or less; a slice that holds a smaller one, other than zero, is left out and contracted on
// the fp32 instruction afterwards, as all of them are where a sum is infinite or NaN (split_tile).  So a result is as good
// as its own terms, whatever larger numbers of its row or column meet zeros.
//
// Lane layout of v_mfma_f32_32x32x16_f16 (lane = 32*h + i): A row i, k = 8*h .. 8*h+7; B column i, the same k; D as
// v_mfma_f32_32x32x2_f32: register r is row 8*(r/4) + 4*h + (r%4), column i.
#pragma once
#include "dn_internal.h"

namespace dn {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
// sixteen bytes at an address that is only a multiple of 4 (rows of odd widths)
typedef float v4f_a4 __attribute__((ext_vector_type(4), aligned(4)));

// BM x BN tile, every wave contracts its own sixteen-k slices (wave w of WK: slices w, w + WK, ...) for the whole
// tile.  Nothing is shared between waves before the partial tiles are added, so the k loop has no barrier: a wave
// keeps two slices of fp32 operands in LDS of its own, filled straight from memory, reads the one that has
// arrived into registers, splits it there and multiplies while the other travels.
// F32: no splitting, the slices go to the fp32 instruction as they are.
template <int BM_, int BN_, int WK_, int OCC_, bool F32_ = false>
struct SliceTile {
    static constexpr bool SPLIT = true, F32 = F32_;
    static constexpr int BM = BM_, BN = BN_, WM = 1, WN = 1, WK = WK_, OCC = OCC_;
    static constexpr int KT = 16 * WK, NT = 64 * WK;
    static constexpr int WTM = BM, WTN = BN, TM = BM / 32, TN = BN / 32;
    static constexpr int STAGE = (BM + BN) * 64;   // bytes of a wave's slice
    static constexpr int BYTES = WK * 2 * STAGE;
};

// One wave's sixteen-k slice of an operand of ROWS rows, fp32 in LDS in pieces of 16 bytes ("slots").
// KC: row r's four pieces at slots 4 r + (c ^ ((r >> 1) & 3)); MC: k's pieces at k ROWS / 4 + (c ^ 8 (k >> 3)) (the
// exclusive-or only for 64 rows).  Both spread the lanes of a read over all banks.
template <bool KC, int ROWS>
struct Slice {
    static constexpr int Q = ROWS / 16;   // slots per lane
    static_assert(ROWS == 32 || ROWS == 64, "rows of a slice");

    // what lane `lane` puts into its q-th slot: row r and k offset k of the piece's first element (four k of a row /
    // four rows of a k)
    static __device__ __forceinline__ void piece(int q, int lane, int &r, int &k)
    {
        const int s = q * 64 + lane;
        if (KC) {
            r = s >> 2;
            k = ((s & 3) ^ ((r >> 1) & 3)) * 4;
        } else {
            k = s / (ROWS / 4);
            r = ((s % (ROWS / 4)) ^ (ROWS == 64 ? (k >> 3) * 8 : 0)) * 4;
        }
    }

    // Byte offsets of the lane's pieces from the slice's first element (leading dimensions are bounded so that they fit
    // 32 bits); rows past the matrix repeat the last piece that lies inside (the products they give are not stored).
    static __device__ __forceinline__ void offsets(unsigned (&off)[Q], int ld, int rows, int lane)
    {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            int r, k;
            piece(q, lane, r, k);
            if (KC) off[q] = ((unsigned)min(r, rows - 1) * (unsigned)ld + (unsigned)k) * 4u;
            else off[q] = ((unsigned)k * (unsigned)ld + (unsigned)min(r, (rows - 4) & ~3)) * 4u;
        }
    }

    // memory -> LDS without registers; sixteen-byte pieces from sixteen-byte aligned addresses, all inside the matrix
    static __device__ __forceinline__ void fetch(const float *slice, const unsigned (&off)[Q], char *lds)
    {
#pragma unroll
        for (int q = 0; q < Q; ++q)
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) unsigned *)(reinterpret_cast<const char *>(slice) + off[q]),
                                             (__attribute__((address_space(3))) unsigned *)(lds + q * 1024), 16, 0, 0);
    }

    // memory -> registers, any alignment; elements outside the matrix are zero
    static __device__ __forceinline__ void load(v4f (&v)[Q], const float *slice, int ld, int rows, int kleft, int lane)
    {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            int r, k;
            piece(q, lane, r, k);
            const float *p = KC ? slice + ((size_t)r * ld + k) : slice + ((size_t)k * ld + r);
            const int first = KC ? kleft - k : rows - r;   // elements of the piece that exist along its own direction
            const bool in = KC ? r < rows : k < kleft;
            if (in && first >= 4) {
                v[q] = *reinterpret_cast<const v4f_a4 *>(p);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[q][j] = (in && j < first) ? p[j] : 0.f;
            }
        }
    }
    static __device__ __forceinline__ void put(char *lds, const v4f (&v)[Q], int lane)
    {
#pragma unroll
        for (int q = 0; q < Q; ++q) *reinterpret_cast<v4f *>(lds + (q * 64 + lane) * 16) = v[q];
    }

    // LDS byte address (from the slice's start) of the lane's operand row of 32-row block b
    static __device__ __forceinline__ void read_at(unsigned (&at)[2], int b, int idx, int h)
    {
        if (KC) {
            const int r = b * 32 + idx, x = (r >> 1) & 3;
            at[0] = (unsigned)(r * 64 + ((2 * h) ^ x) * 16);
            at[1] = (unsigned)(r * 64 + ((2 * h + 1) ^ x) * 16);
        } else {
            const int r = ROWS == 64 ? (b * 32 + idx) ^ (h * 32) : b * 32 + idx;
            at[0] = at[1] = (unsigned)(h * 8 * ROWS * 4 + r * 4);
        }
    }
};

// The eight k values of the lane's row in each block.  The wait is part of the statement: the compiler does not know
// that these read memory that fetch() fills, and must not use (or reuse) the registers before they have arrived.
template <bool KC, int ROWS>
__device__ __forceinline__ void read_blocks(v4f (&x)[ROWS / 32][2], unsigned base, const unsigned (&at)[ROWS / 32][2])
{
    if (KC) {
        if (ROWS == 64)
            asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
                         "s_waitcnt lgkmcnt(0)"
                         : "=&v"(x[0][0]), "=&v"(x[0][1]), "=&v"(x[ROWS / 32 - 1][0]), "=&v"(x[ROWS / 32 - 1][1])
                         : "v"(base + at[0][0]), "v"(base + at[0][1]), "v"(base + at[ROWS / 32 - 1][0]), "v"(base + at[ROWS / 32 - 1][1])
                         : "memory");
        else
            asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                         : "=&v"(x[0][0]), "=&v"(x[0][1]) : "v"(base + at[0][0]), "v"(base + at[0][1]) : "memory");
    } else if (ROWS == 64) {
        v2f p[8];
        asm volatile("ds_read2st64_b32 %0, %8 offset0:0 offset1:1\n\tds_read2st64_b32 %1, %8 offset0:2 offset1:3\n\t"
                     "ds_read2st64_b32 %2, %8 offset0:4 offset1:5\n\tds_read2st64_b32 %3, %8 offset0:6 offset1:7\n\t"
                     "ds_read2st64_b32 %4, %9 offset0:0 offset1:1\n\tds_read2st64_b32 %5, %9 offset0:2 offset1:3\n\t"
                     "ds_read2st64_b32 %6, %9 offset0:4 offset1:5\n\tds_read2st64_b32 %7, %9 offset0:6 offset1:7\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(p[0]), "=&v"(p[1]), "=&v"(p[2]), "=&v"(p[3]), "=&v"(p[4]), "=&v"(p[5]), "=&v"(p[6]), "=&v"(p[7])
                     : "v"(base + at[0][0]), "v"(base + at[ROWS / 32 - 1][0]) : "memory");
#pragma unroll
        for (int i = 0; i < ROWS / 32; ++i) {
            x[i][0] = (v4f){p[i * 4][0], p[i * 4][1], p[i * 4 + 1][0], p[i * 4 + 1][1]};
            x[i][1] = (v4f){p[i * 4 + 2][0], p[i * 4 + 2][1], p[i * 4 + 3][0], p[i * 4 + 3][1]};
        }
    } else {
        v2f p[4];
        asm volatile("ds_read2_b32 %0, %4 offset0:0 offset1:32\n\tds_read2_b32 %1, %4 offset0:64 offset1:96\n\t"
                     "ds_read2_b32 %2, %4 offset0:128 offset1:160\n\tds_read2_b32 %3, %4 offset0:192 offset1:224\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(p[0]), "=&v"(p[1]), "=&v"(p[2]), "=&v"(p[3]) : "v"(base + at[0][0]) : "memory");
        x[0][0] = (v4f){p[0][0], p[0][1], p[1][0], p[1][1]};
        x[0][1] = (v4f){p[2][0], p[2][1], p[3][0], p[3][1]};
    }
}

// scale x = h + 2^-11 l, both f16.
__device__ __forceinline__ void split_eight(const v4f &lo, const v4f &hi, float scale, v8h (&f)[2])
{
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float x0 = q < 2 ? lo[2 * q] : hi[2 * q - 4], x1 = q < 2 ? lo[2 * q + 1] : hi[2 * q - 3];
        const v2h h = __builtin_convertvector((v2f){x0 * scale, x1 * scale}, v2h);
        const float r0 = __builtin_fmaf(x0, scale, -(float)h[0]), r1 = __builtin_fmaf(x1, scale, -(float)h[1]);
        const v2h l = __builtin_convertvector((v2f){r0 * 2048.f, r1 * 2048.f}, v2h);
        f[0][2 * q] = h[0];
        f[0][2 * q + 1] = h[1];
        f[1][2 * q] = l[0];
        f[1][2 * q + 1] = l[1];
    }
}

// Largest and smallest magnitude of eight numbers.  (fmaxf and fminf would each quiet their operands first.)
__device__ __forceinline__ float max3_magnitude(float a, float b, float c)
{
    float m;
    asm("v_max3_f32 %0, |%1|, |%2|, |%3|" : "=v"(m) : "v"(a), "v"(b), "v"(c));
    return m;
}
__device__ __forceinline__ float min3_magnitude(float a, float b, float c)
{
    float m;
    asm("v_min3_f32 %0, |%1|, |%2|, |%3|" : "=v"(m) : "v"(a), "v"(b), "v"(c));
    return m;
}
__device__ __forceinline__ float largest(const v4f &lo, const v4f &hi)
{
    return max3_magnitude(max3_magnitude(lo[0], lo[1], lo[2]), max3_magnitude(lo[3], hi[0], hi[1]), max3_magnitude(hi[2], hi[3], hi[3]));
}
__device__ __forceinline__ float smallest(const v4f &lo, const v4f &hi)
{
    return min3_magnitude(min3_magnitude(lo[0], lo[1], lo[2]), min3_magnitude(lo[3], hi[0], hi[1]), min3_magnitude(hi[2], hi[3], hi[3]));
}

// The smallest magnitude among eight numbers that are not zero, as twice its bits less one.  (Shifted left the sign is
// gone, and less one a zero is the largest of unsigned numbers.)
__device__ __forceinline__ unsigned magnitude_key(float x) { return (__float_as_uint(x) << 1) - 1u; }
__device__ __forceinline__ unsigned least_key(const v4f &lo, const v4f &hi)
{
    unsigned m = ~0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) m = min(min(m, magnitude_key(lo[q])), magnitude_key(hi[q]));
    return m;
}

}  // namespace dn

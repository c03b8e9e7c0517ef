// The filter gradient of 3 x 3, stride-1 layers with wide channels, eight images to a lane (included by dn_conv.hip, which has
// ConvShape and the plan).
#ifndef DN_CONV_DW_H
#define DN_CONV_DW_H

namespace dn {
namespace {

// dW[oc][ic][tap] = sum over images and pixels of delta[image][oc][pixel] x[image][ic][pixel + tap] (the divisor and the order of
// the chunks are conv_dw_reduce_kernel's).  Per tap it is a product whose long edge, images x pixels, is not contiguous in either
// operand for a fixed channel, and shifts by the tap in one of them.  Here the eight numbers a lane puts into a matrix instruction
// (k) are the same pixel of eight images, and its lower and upper half of the lanes hold two neighbouring pixels: a tap then moves a
// lane's address by whole 16-byte words, and no operand is ever read across a word.
//
// Numbers are kept as three bf16 parts, each what is left rounded to nearest (v = h + m + l exactly): six products, hh hm mh mm hl lh,
// leave out terms of 2^-25 of the product and less, of either sign.  Three parts need no scale and no test of what fits beside the largest
// (two f16 parts would take three products, but deltas span more than their range).  What is not finite, or rounds to infinity, spoils the
// sum it enters, and a number below 2^-110 may have a last bit below 2^-133, bf16's smallest number (the instruction keeps subnormal numbers:
// 2^-133 times 2^97 is 2^-36, and a product of 2^-133 is one): a workgroup that has found the first when it has finished, or meets the
// second on its way, goes through its pixels with fp32 operands on the fp32 instruction instead.  (The layer pair below 150 us; with one
// such small number an image 191, 214 with the first pass finished, 181 all in fp32; deltas of 1e-35 195, 225 and 196.)
// The bf16 instruction rounds its sums downwards.  So no long sum is formed on it: sixteen products at a time (six instructions, the
// small terms first) begin at zero and are added to the long sum on the vector unit, to nearest; and pixels 4..7 and 12..15 of a row
// enter with their sign turned and their sums are subtracted.  Errors of dW against 64 bits (1e-8; fp32 instruction / long sums on the
// bf16 instruction, parts cut off / this): 128 images of 32 x 32, 32 -> 64 channels, normal numbers 35 / 21 / 14, with ReLU on the input
// 27 / 21 / 14, all positive 6.4 / 7.2 / 5.9; 256 images of 48 x 24, 64 -> 128 81 / 60 / 20, 58 / 59 / 20, 8.2 / 82 / 5.5.
//
// A workgroup of eight waves owns 64 output x 32 input channels, all nine taps, and a run of the rows [8 images][16 columns]
// (rows in the order image group, strip of columns, row).  LDS holds the row's delta and three rows of the input (the next input
// row takes the place of the oldest), requested a row ahead.  Wave (o, q) takes output channels 32 o .. and pixels 4 q .. 4 q + 3:
// nine accumulator tiles, 108 matrix instructions for 51 reads of 16 bytes a row.  The four q are added through LDS at the end.
// The slot of channel c at pixel p is (c + p) mod 32 (64): writes, whose lanes run over pixels, and reads, whose lanes run over
// channels, both spread over all banks.
// Bound: the matrix unit half of the time; storing the parts and requesting the next row, in which all waves move together; 16 additions
// for six matrix instructions, beside the other wave's.  128 images 32 x 32 x 32 -> 64: 44 us (52 to 66 on the fp32 instruction, by what
// runs before it; 39 with the long sums on the bf16 instruction).  With the delta pass: 60 (82; 55); requests between the products spill (17 registers,
// slower); sums of both pixel pairs of a tap before they are added: 20 reloads a row, 64; two short sums at a time, one added while the other
// is formed: 18 to 39 reloads, 63 to 77.
constexpr int DWI_THREADS = 512, DWI_TW = 16, DWI_XW = DWI_TW + 2, DWI_IMAGES = 8, DWI_OC = 64, DWI_IC = 32;
constexpr int DWI_XROW = DWI_XW * DWI_IC * 16, DWI_XPART = 3 * DWI_XROW, DWI_DPART = DWI_TW * DWI_OC * 16;   // bytes
constexpr int DWI_STAGE = 3 * (DWI_XPART + DWI_DPART), DWI_SUMS = 4 * 9 * 16 * 64 * 4;
constexpr int DWI_LDS = DWI_SUMS > DWI_STAGE + 16 ? DWI_SUMS : DWI_STAGE + 16;

typedef __bf16 v8b_t __attribute__((ext_vector_type(8)));
typedef unsigned v4u_t __attribute__((ext_vector_type(4)));
typedef float v4s_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned two_bf16(float lo, float hi)   // rounded to nearest
{
    typedef __bf16 v2b __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(unsigned, v2b{(__bf16)lo, (__bf16)hi});
}

// eight numbers of one channel and pixel into LDS: as three bf16 parts or (FP32) as two 16-byte words; least: twice the bits of the
// smallest magnitude that is not zero, less one
constexpr unsigned DWI_LEAST = (18u << 24) - 1u;   // of 2^-109: a smaller one's last bits may be less than bf16 holds
template <bool FP32>
__device__ __forceinline__ void dwi_store(const float (&v)[8], char *at, int part, unsigned &least)
{
    if constexpr (FP32) {
#pragma unroll
        for (int w = 0; w < 2; ++w) *reinterpret_cast<v4s_t *>(at + w * part) = v4s_t{v[4 * w], v[4 * w + 1], v[4 * w + 2], v[4 * w + 3]};
    } else {
        v4u_t p[3];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float a = v[2 * j], b = v[2 * j + 1];
            p[0][j] = two_bf16(a, b);
            const float a1 = a - __uint_as_float(p[0][j] << 16), b1 = b - __uint_as_float(p[0][j] & 0xffff0000u);
            p[1][j] = two_bf16(a1, b1);
            p[2][j] = two_bf16(a1 - __uint_as_float(p[1][j] << 16), b1 - __uint_as_float(p[1][j] & 0xffff0000u));
            least = min(least, min((__float_as_uint(a) << 1) - 1u, (__float_as_uint(b) << 1) - 1u));
        }
#pragma unroll
        for (int w = 0; w < 3; ++w) *reinterpret_cast<v4u_t *>(at + w * part) = p[w];
    }
}

// One workgroup's rows lo .. hi - 1: accumulators (added to) and the sums of the delta values this thread stages (set).  False, for
// all threads: a row has a number too small for its parts, and it and the rows behind it have been left.
template <bool FP32>
__device__ __forceinline__ bool dwi_rows(const ConvShape &s, const float *__restrict__ X, const float *__restrict__ delta, int ic0,
                                         int oc0, int lo, int hi, int strips, char *lds, v16f_t (&acc)[9], float (&bsum)[2])
{
    constexpr int PARTS = FP32 ? 2 : 3;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, idx = lane & 31, h = lane >> 5;
    const int o = wave & 1, q = wave >> 1;
    char *xs = lds, *ds = lds + 3 * DWI_XPART;
    volatile int *too_small = reinterpret_cast<volatile int *>(lds + DWI_STAGE);
    if (!FP32 && tid == 0) *too_small = 0;   // (read behind two barriers)
    const unsigned pix = (unsigned)(s.Ho * s.Wo), in = (unsigned)(s.H * s.W);
    // what this thread stages: delta of two output channels and the input of one channel at one column; the first wave also the two
    // last columns of the input
    const int sp = tid & 15, sc = tid >> 4, hp = 16 + (tid & 1), hc = (tid & 63) >> 1;
    const bool halo = tid < 64;
    const unsigned d_at[2] = {(unsigned)min(oc0 + sc, s.Cout - 1) * pix, (unsigned)min(oc0 + 32 + sc, s.Cout - 1) * pix};
    const unsigned x_at = (unsigned)min(ic0 + sc, s.Cin - 1) * in, h_at = (unsigned)min(ic0 + hc, s.Cin - 1) * in;
    const bool d_on[2] = {oc0 + sc < s.Cout, oc0 + 32 + sc < s.Cout}, x_on = ic0 + sc < s.Cin, h_on = ic0 + hc < s.Cin;
    char *d_to[2], *x_to = xs + sp * (DWI_IC * 16) + ((sc + sp) & 31) * 16, *h_to = xs + hp * (DWI_IC * 16) + ((hc + hp) & 31) * 16;
#pragma unroll
    for (int k = 0; k < 2; ++k) d_to[k] = ds + sp * (DWI_OC * 16) + ((sc + 32 * k + sp) & 63) * 16;
    // what it multiplies
    const char *a_from[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int p = 4 * q + 2 * k + h;
        a_from[k] = ds + p * (DWI_OC * 16) + ((32 * o + idx + p) & 63) * 16;
    }
    const char *b_from = xs + (4 * q + h) * (DWI_IC * 16);
    const int b_slot = idx + 4 * q + h;
    const unsigned turned = sp & 4 ? 0x80000000u : 0u;
    bsum[0] = bsum[1] = 0.f;

    // Loads are unconditional, from an address clamped into the tensor; what lies outside becomes zero as it is stored.
    // (An image's bytes fit 31 bits: takes_images.)
    const char *x_base[8], *d_base[8];   // of the eight images
    auto images_from = [&](int first) {
        const size_t x_image = (size_t)s.Cin * in * 4, d_image = (size_t)s.Cout * pix * 4;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const size_t b = (size_t)min(first + j, s.B - 1);
            x_base[j] = reinterpret_cast<const char *>(X) + b * x_image;
            d_base[j] = reinterpret_cast<const char *>(delta) + b * d_image;
        }
    };
    auto load = [&](const char *const (&base)[8], unsigned off, float (&v)[8]) {
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const float *>(base[j] + off * 4u);
    };
    auto x_off = [&](unsigned at, int y, int col) {   // patch row y (image row y - pad), image column col - pad
        return at + (unsigned)min(max(y - s.pad, 0), s.H - 1) * (unsigned)s.W + (unsigned)min(max(col - s.pad, 0), s.W - 1);
    };
    auto blank = [&](float (&v)[8], bool on, int images) {
        if (images >= 8 && __all(on)) return;
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = on && j < images ? v[j] : 0.f;
    };
    struct Row { int first, x0, y; };
    auto row_of = [&](int r) {
        const int line = r / s.Ho;
        return Row{line / strips * DWI_IMAGES, line % strips * DWI_TW, r % s.Ho};
    };
    float dv[2][8], xv[8], hv[8];
    // a row's delta and the input row two below its first tap row, in three portions
    auto fetch = [&](const Row &r, int portion) {
        if (portion < 2) load(d_base, d_at[portion] + (unsigned)r.y * (unsigned)s.Wo + (unsigned)min(r.x0 + sp, s.Wo - 1), dv[portion]);
        else {
            load(x_base, x_off(x_at, r.y + 2, r.x0 + sp), xv);
            if (halo) load(x_base, x_off(h_at, r.y + 2, r.x0 + hp), hv);
        }
    };
    auto put_x = [&](const Row &r, int y, float (&a)[8], float (&b)[8], unsigned &least) {
        const bool row_on = y >= s.pad && y - s.pad < s.H;
        const int images = s.B - r.first, to = y % 3 * DWI_XROW;
        auto col_on = [&](int col) { return col >= s.pad && col - s.pad < s.W; };
        blank(a, row_on && x_on && col_on(r.x0 + sp), images);
        dwi_store<FP32>(a, x_to + to, DWI_XPART, least);
        if (halo) {
            blank(b, row_on && h_on && col_on(r.x0 + hp), images);
            dwi_store<FP32>(b, h_to + to, DWI_XPART, least);
        }
    };

    Row r = row_of(lo);
    for (int n = lo; n < hi; ++n) {
        unsigned least = ~0u;
        const bool fresh = n == lo || r.y == 0;   // the two upper tap rows are not in LDS, and nothing has been requested
        if (fresh) {
            images_from(r.first);
#pragma unroll
            for (int k = 0; k < 2; ++k) load(x_base, x_off(x_at, r.y + k, r.x0 + sp), dv[k]);
            if (halo) {
                load(x_base, x_off(h_at, r.y, r.x0 + hp), xv);
                load(x_base, x_off(h_at, r.y + 1, r.x0 + hp), hv);
            }
        }
        __syncthreads();   // the previous row has been used
        if (fresh) {
            put_x(r, r.y, dv[0], xv, least);
            put_x(r, r.y + 1, dv[1], hv, least);
#pragma unroll
            for (int k = 0; k < 3; ++k) fetch(r, k);
        }
        put_x(r, r.y + 2, xv, hv, least);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            blank(dv[k], d_on[k] && r.x0 + sp < s.Wo, s.B - r.first);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                bsum[k] += dv[k][j];
                dv[k][j] = __uint_as_float(__float_as_uint(dv[k][j]) ^ turned);
            }
            dwi_store<FP32>(dv[k], d_to[k], DWI_DPART, least);
        }
        if (!FP32 && least < DWI_LEAST) *too_small = 1;
        __syncthreads();
        if (!FP32 && *too_small) return false;   // (set again behind the next barrier at the earliest)
        const int y = r.y;
        r = row_of(n + 1);
        if (n + 1 < hi && r.y > 0) {
#pragma unroll
            for (int k = 0; k < 3; ++k) fetch(r, k);
        }
// step e = 9 k + 3 ky + kx: pixels 2 k + h, whose input pixels for tap kx are kx + 2 k + h
        v4u_t a[PARTS], b[2][PARTS];
        auto b_load = [&](int e) {
            const int d = e % 3 + 2 * (e / 9);
            const char *b_at = b_from + (y + e / 3 % 3) % 3 * DWI_XROW + d * (DWI_IC * 16) + ((b_slot + d) & 31) * 16;
#pragma unroll
            for (int w = 0; w < PARTS; ++w) b[e & 1][w] = *reinterpret_cast<const v4u_t *>(b_at + w * DWI_XPART);
        };
        b_load(0);
#pragma unroll
        for (int e = 0; e < 18; ++e) {
            if (e % 9 == 0) {
#pragma unroll
                for (int w = 0; w < PARTS; ++w) a[w] = *reinterpret_cast<const v4u_t *>(a_from[e / 9] + w * DWI_DPART);
            }
            if (e < 17) b_load(e + 1);
            v16f_t &c = acc[e % 9];
            if constexpr (FP32) {
#pragma unroll
                for (int j = 0; j < 8; ++j)
                    c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[j >> 2][j & 3]), __uint_as_float(b[e & 1][j >> 2][j & 3]), c, 0, 0, 0);
            } else {
                v16f_t t = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                auto mul = [&](int u, int v) {
                    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(v8b_t, a[u]), __builtin_bit_cast(v8b_t, b[e & 1][v]), t, 0, 0, 0);
                };
                mul(2, 0); mul(0, 2); mul(1, 1); mul(1, 0); mul(0, 1); mul(0, 0);
#pragma unroll
                for (int i = 0; i < 16; ++i) c[i] += t[i];
                asm volatile("" : "+v"(c));   // (stays where it is: without this the allocator moves and spills the nine)
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    return true;
}

// grid: (input groups of 32 x output groups of 64, chunks).  part[chunk]: filter sums as [tap][oc][ic], then the bias sums.
__global__ __launch_bounds__(DWI_THREADS, 2) void conv_dw_images_kernel(ConvShape s, const float *__restrict__ X,
                                                                        const float *__restrict__ delta, float *__restrict__ part,
                                                                        int strips, int rows)
{
    __shared__ __attribute__((aligned(16))) char lds[DWI_LDS];
    const int groups = (s.Cin + DWI_IC - 1) / DWI_IC;
    const int ic0 = (int)(blockIdx.x % groups) * DWI_IC, oc0 = (int)(blockIdx.x / groups) * DWI_OC;
    const int lo = (int)((long)rows * blockIdx.y / gridDim.y), hi = (int)((long)rows * (blockIdx.y + 1) / gridDim.y);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, idx = lane & 31, h = lane >> 5, o = wave & 1, q = wave >> 1;
    v16f_t acc[9];
    float bsum[2];
    // (0 + 2) - (1 + 3) of the four q: the upper two leave theirs in LDS, then q 0 and 1 exchange what the other one finishes
    auto at = [&](int w, int t, int i) { return reinterpret_cast<v4s_t *>(lds + (((w * 9 + t) * 4 + i) * 64 + lane) * 16); };
    auto put = [&](int w, int t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) *at(w, t, i) = v4s_t{acc[t][4 * i], acc[t][4 * i + 1], acc[t][4 * i + 2], acc[t][4 * i + 3]};
    };
    auto add = [&](int w, int t, bool more) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const v4s_t v = *at(w, t, i);
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[t][4 * i + j] = more ? acc[t][4 * i + j] + v[j] : acc[t][4 * i + j] - v[j];
        }
    };
    auto clear = [&] {
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[t][i] = 0.f;
    };
    auto merge = [&] {   // whether all sums are finite
        __syncthreads();
        if (q >= 2) {
#pragma unroll
            for (int t = 0; t < 9; ++t) put(wave - 4, t);
        }
        __syncthreads();
        if (q < 2) {
#pragma unroll
            for (int t = 0; t < 9; ++t) add(wave, t, true);
#pragma unroll
            for (int t = 0; t < 9; ++t)
                if ((t < 5) == (q == 1)) put(wave, t);   // over what this wave has just read
        }
        __syncthreads();
        float zero = 0.f;
        if (q < 2) {
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                if ((t < 5) != (q == 0)) continue;
                add(wave ^ 2, t, false);
#pragma unroll
                for (int i = 0; i < 16; ++i) zero = fmaf(acc[t][i], 0.f, zero);   // NaN where a sum is not finite
            }
        }
        return !__syncthreads_or(!(zero == 0.f));
    };
    clear();
    if (!dwi_rows<false>(s, X, delta, ic0, oc0, lo, hi, strips, lds, acc, bsum) || !merge()) {
        clear();
        dwi_rows<true>(s, X, delta, ic0, oc0, lo, hi, strips, lds, acc, bsum);
        merge();
    }
    const size_t plane = (size_t)s.Cout * s.Cin, filt = 9 * plane;
    float *out = part + (size_t)blockIdx.y * (filt + s.Cout);
    if (q < 2) {
        const bool whole = oc0 + DWI_OC <= s.Cout && ic0 + DWI_IC <= s.Cin;
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            if ((t < 5) != (q == 0)) continue;
            float *to = out + t * plane + (size_t)(oc0 + 32 * o + 4 * h) * s.Cin + ic0 + idx;
            if (whole) {
#pragma unroll
                for (int i = 0; i < 16; ++i) to[(size_t)(8 * (i >> 2) + (i & 3)) * s.Cin] = q == 0 ? acc[t][i] : -acc[t][i];
            } else {
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int oc = oc0 + 32 * o + 8 * (i >> 2) + 4 * h + (i & 3);
                    if (oc < s.Cout && ic0 + idx < s.Cin) to[(size_t)(8 * (i >> 2) + (i & 3)) * s.Cin] = q == 0 ? acc[t][i] : -acc[t][i];
                }
            }
        }
    }
    if (ic0 == 0) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            float b = bsum[k];
#pragma unroll
            for (int m = 8; m >= 1; m >>= 1) b += __shfl_xor(b, m);
            const int oc = oc0 + 32 * k + (int)(threadIdx.x >> 4);
            if ((threadIdx.x & 15) == 0 && oc < s.Cout) out[filt + oc] = b;
        }
    }
}

}  // namespace
}  // namespace dn

#endif

// kf_quant.hip -- row-scaled reduced-precision storage of an FP32 matrix (the
// storage kf_matrix_q declares): BF16 with scale 1, or OCP FP8-E4M3 with one
// FP32 scale per row, scale_i = amax_i / 448 (448 is the largest finite E4M3
// value). Every code is the nearest value, ties to even, of the exact number
// it stands for (a_ij for BF16, the exact quotient a_ij / scale_i for FP8),
// with FP8 saturating at +-448.
#include <hip/hip_runtime.h>

#include <cstdint>

namespace kf {
namespace {

// BF16: round the binary32 value to 8 significant bits, ties to even (adding
// 0x7fff plus the kept lowest bit carries exactly when the dropped half is
// above one half, or equal to it with an odd kept part). NaN stays a quiet NaN.
__device__ __forceinline__ unsigned short bf16_code(float x) {
    const unsigned u = __float_as_uint(x);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (unsigned short)((u >> 16) | 0x40u);
    return (unsigned short)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

// Magnitude of E4M3 code c (0 <= c <= 0x7e): c = e << 3 | m stands for
// m 2^-9 when e = 0 and (1 + m / 8) 2^(e - 7) otherwise.
__device__ __forceinline__ float e4m3_mag(unsigned c) {
    const unsigned e = c >> 3, m = c & 7u;
    return e == 0 ? (float)m * 0x1p-9f : __uint_as_float(((e + 120u) << 23) | (m << 20));
}

// E4M3 code of x / s (s > 0 finite). q = x / s in binary32 is within a few
// units in the last place of the exact quotient, far less than half the E4M3
// spacing, so its neighbours lo <= |q| < hi on the E4M3 grid bracket the exact
// quotient or the exact quotient lies within those few units of one of them
// (then that one is the nearest). The choice between lo and hi compares
// |x| with mid s, mid = (lo + hi) / 2 exact in binary32, by the sign of one
// fused multiply-add, so it is exact; both operands are first scaled by 2^64
// when s is small so that the difference cannot underflow to zero.
__device__ __forceinline__ unsigned char e4m3_code(float x, float s) {
    const unsigned sign = (__float_as_uint(x) >> 24) & 0x80u;
    if (x != x) return (unsigned char)(sign | 0x7fu);
    const float a = fabsf(x / s);
    if (!(a < 448.f)) return (unsigned char)(sign | 0x7eu);   // saturate (includes +inf)
    unsigned lo;
    if (a < 0x1p-6f) {
        lo = (unsigned)(a * 0x1p9f);                 // subnormal grid m 2^-9 (exact scaling)
    } else {
        const unsigned b = __float_as_uint(a);
        lo = ((((b >> 23) - 127u + 7u) << 3) | ((b >> 20) & 7u));
    }
    const float vlo = e4m3_mag(lo);
    if (vlo == a) return (unsigned char)(sign | lo);
    const float vhi = e4m3_mag(lo + 1u);
    const float mid = 0.5f * (vlo + vhi);
    const float k = s < 0x1p-60f ? 0x1p64f : 1.f;
    const float r = __builtin_fmaf(-mid, s * k, fabsf(x) * k);
    unsigned c;
    if (r > 0.f) c = lo + 1u;
    else if (r < 0.f) c = lo;
    else c = (lo & 1u) ? lo + 1u : lo;              // tie: the even code
    return (unsigned char)(sign | c);
}

// Rows are walked in chunks of four consecutive elements, one 16-byte load and
// one 4-byte (FP8) or 8-byte (BF16) store per lane, so a wave reads 1 KiB and
// writes whole 128-byte lines. T lanes share a row and chunk c belongs to lane
// c mod T; the K first chunks of each lane stay in registers between the row
// maximum and the conversion, so rows of up to 4 T K columns are read once.
typedef float f4 __attribute__((ext_vector_type(4)));
// FP32 rows start at any multiple of 4 bytes; global loads of 16 bytes need no more.
typedef f4 f4_any __attribute__((aligned(4)));
typedef unsigned u2 __attribute__((ext_vector_type(2)));

// Columns 4 c .. 4 c + 3 of a row (zero at and past `cols`).
__device__ __forceinline__ f4 load_chunk(const float* a, long c, long cols) {
    const long j = 4 * c;
    if (j + 4 <= cols) return __builtin_nontemporal_load(reinterpret_cast<const f4_any*>(a + j));
    f4 v = {0.f, 0.f, 0.f, 0.f};
    if (j + 0 < cols) v.x = a[j + 0];
    if (j + 1 < cols) v.y = a[j + 1];
    if (j + 2 < cols) v.z = a[j + 2];
    return v;
}
__device__ __forceinline__ unsigned mag_bits(f4 v, unsigned m) {
    m = max(m, __float_as_uint(v.x) & 0x7fffffffu);
    m = max(m, __float_as_uint(v.y) & 0x7fffffffu);
    m = max(m, __float_as_uint(v.z) & 0x7fffffffu);
    return max(m, __float_as_uint(v.w) & 0x7fffffffu);
}
__device__ __forceinline__ unsigned pack_fp8(f4 v) {   // hardware rounding to nearest even
    int w = __builtin_amdgcn_cvt_pk_fp8_f32(v.x, v.y, 0, false);
    return (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(v.z, v.w, w, true);
}
__device__ __forceinline__ unsigned exact_fp8(f4 v, float s) {
    return (unsigned)e4m3_code(v.x, s) | (unsigned)e4m3_code(v.y, s) << 8 | (unsigned)e4m3_code(v.z, s) << 16 |
           (unsigned)e4m3_code(v.w, s) << 24;
}
// Four codes of v / s. lo and hi are reciprocals of s a little below and above
// 1 / s: the exact quotient lies between v lo and v hi (their own rounding
// included), rounding to E4M3 is monotone, so equal codes of the two products
// are the code of the exact quotient. They differ only within 2^-20 of a
// rounding boundary (about one chunk in 10^4); those take the exact route.
__device__ __forceinline__ unsigned fp8_codes(f4 v, float s, float lo, float hi) {
    const unsigned a = pack_fp8(v * lo), b = pack_fp8(v * hi);
    return __builtin_expect(a == b, 1) ? a : exact_fp8(v, s);
}
__device__ __forceinline__ u2 bf16_codes(f4 v) {
    u2 w;
    w.x = (unsigned)bf16_code(v.x) | (unsigned)bf16_code(v.y) << 16;
    w.y = (unsigned)bf16_code(v.z) | (unsigned)bf16_code(v.w) << 16;
    return w;
}

// Bounds on the row scale for the products above: 1 / s, v lo and v hi stay
// normal for every quotient that does not round to zero, and the largest
// quotient 448 (1 + 2^-24) still rounds to 448. Rows with other scales, and
// rows that hold an infinity or a NaN, take the exact route throughout.
constexpr float kScaleLo = 0x1p-100f, kScaleHi = 0x1p100f;

// T lanes per row, K chunks per lane in registers, 256 / T rows per workgroup
// (one row of T lanes when T >= 256). Bound by the HBM streams (4 bytes in, 1 or
// 2 out per element): 8192 x 8192 to FP8 takes 56.5 us, 5.9 TB/s of those bytes,
// against 169.5 us when each row was read twice by 4-byte loads, coded by the
// exact route alone (about 45 VALU operations an element against 6) and stored
// by single bytes.
template <int FP8, int T, int K>
__global__ void __launch_bounds__(T > 256 ? T : 256)
kf_quantize_rows_kernel(const float* __restrict__ A, long rows, long cols, long lda, void* __restrict__ codes, long ldq,
                        float* __restrict__ scales) {
    constexpr int NT = T > 256 ? T : 256, RPB = NT / T;
    const int t = threadIdx.x % T;
    const long i = (long)blockIdx.x * RPB + threadIdx.x / T;
    if (RPB > 1 && i >= rows) return;   // whole waves (T is 64): no barrier below
    const float* a = A + i * lda;
    const long nc = (cols + 3) / 4, nq = ldq / 4;   // chunks that hold data, chunks of the stored row
    f4 v[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        v[k] = f4{0.f, 0.f, 0.f, 0.f};
        if (t + (long)k * T < nc) v[k] = load_chunk(a, t + (long)k * T, cols);
    }
    float s = 1.f;
    if constexpr (FP8) {
        // the largest magnitude as an integer: above 0x7f800000 the row holds a NaN
        unsigned m = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) m = mag_bits(v[k], m);
        for (long c = t + (long)K * T; c < nc; c += T) m = mag_bits(load_chunk(a, c, cols), m);
        for (int o = 32; o > 0; o >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, o));
        if constexpr (T > 64) {
            __shared__ unsigned red[T / 64];
            if ((t & 63) == 0) red[t >> 6] = m;
            __syncthreads();
#pragma unroll
            for (int w = 0; w < T / 64; ++w) m = max(m, red[w]);
        }
        float amax = __uint_as_float(m);
        if (m > 0x7f800000u) {   // NaN entries do not count: the row again, by value
            amax = 0.f;
            for (long j = t; j < cols; j += T) amax = fmaxf(amax, fabsf(a[j]));
            for (int o = 32; o > 0; o >>= 1) amax = fmaxf(amax, __shfl_xor(amax, o));
            if constexpr (T > 64) {
                __shared__ float redf[T / 64];
                if ((t & 63) == 0) redf[t >> 6] = amax;
                __syncthreads();
#pragma unroll
                for (int w = 0; w < T / 64; ++w) amax = fmaxf(amax, redf[w]);
            }
        }
        if (amax > 0.f && amax <= 3.4028235e38f) s = __fdiv_rn(amax, 448.f);
        if (t == 0) scales[i] = s;
        unsigned* q = reinterpret_cast<unsigned*>(static_cast<unsigned char*>(codes) + i * ldq);
        if (m <= 0x7f7fffffu && s >= kScaleLo && s <= kScaleHi) {
            const float inv = __fdiv_rn(1.f, s), lo = inv * (1.f - 0x1p-21f), hi = inv * (1.f + 0x1p-21f);
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (t + (long)k * T < nq) __builtin_nontemporal_store(fp8_codes(v[k], s, lo, hi), q + t + (long)k * T);
            for (long c = t + (long)K * T; c < nq; c += T)
                __builtin_nontemporal_store(fp8_codes(load_chunk(a, c, cols), s, lo, hi), q + c);
        } else {
            for (long c = t; c < nq; c += T) q[c] = exact_fp8(load_chunk(a, c, cols), s);
        }
    } else {
        if (t == 0) scales[i] = s;
        u2* q = reinterpret_cast<u2*>(static_cast<unsigned short*>(codes) + i * ldq);
#pragma unroll
        for (int k = 0; k < K; ++k)
            if (t + (long)k * T < nq) __builtin_nontemporal_store(bf16_codes(v[k]), q + t + (long)k * T);
        for (long c = t + (long)K * T; c < nq; c += T) __builtin_nontemporal_store(bf16_codes(load_chunk(a, c, cols)), q + c);
    }
}

template <int FP8, int T, int K>
hipError_t launch(const float* A, long rows, long cols, long lda, void* codes, long ldq, float* scales, hipStream_t st) {
    constexpr int NT = T > 256 ? T : 256, RPB = NT / T;
    // a launch has fewer than 2^32 threads: 4194303 rows of 1024 lanes
    constexpr long most = ((1L << 32) - 1) / NT * RPB;
    for (long r = 0; r < rows; r += most) {
        const long n = rows - r < most ? rows - r : most;
        hipLaunchKernelGGL((kf_quantize_rows_kernel<FP8, T, K>), dim3((unsigned)((n + RPB - 1) / RPB)), dim3(NT), 0, st,
                           A + r * lda, n, cols, lda, static_cast<char*>(codes) + r * ldq * (FP8 ? 1 : 2), ldq, scales + r);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Lanes per row and chunks per lane: the fewest lanes that hold the row in
// registers, a wave up to 2048 columns, 256 lanes up to 8192, 1024 lanes up to
// 32768; wider rows read what the registers do not hold a second time.
template <int FP8>
hipError_t launch_fmt(const float* A, long rows, long cols, long lda, void* codes, long ldq, float* scales, hipStream_t st) {
    if (cols <= 64 * 4 * 2) return launch<FP8, 64, 2>(A, rows, cols, lda, codes, ldq, scales, st);
    if (cols <= 64 * 4 * 4) return launch<FP8, 64, 4>(A, rows, cols, lda, codes, ldq, scales, st);
    if (cols <= 64 * 4 * 8) return launch<FP8, 64, 8>(A, rows, cols, lda, codes, ldq, scales, st);
    if (cols <= 256 * 4 * 4) return launch<FP8, 256, 4>(A, rows, cols, lda, codes, ldq, scales, st);
    if (cols <= 256 * 4 * 8) return launch<FP8, 256, 8>(A, rows, cols, lda, codes, ldq, scales, st);
    if (cols <= 1024 * 4 * 4) return launch<FP8, 1024, 4>(A, rows, cols, lda, codes, ldq, scales, st);
    return launch<FP8, 1024, 8>(A, rows, cols, lda, codes, ldq, scales, st);
}

}  // namespace

hipError_t launch_quantize_rows(const float* A, long rows, long cols, long lda, int fp8, void* codes, long ldq,
                                float* scales, hipStream_t st) {
    if (rows <= 0) return hipSuccess;
    return fp8 ? launch_fmt<1>(A, rows, cols, lda, codes, ldq, scales, st)
               : launch_fmt<0>(A, rows, cols, lda, codes, ldq, scales, st);
}

}  // namespace kf

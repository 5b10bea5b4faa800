// kf_batch.hip -- one persistent launch over many uneven-size BiCGK and GEMVER
// instances.
//
// The paper fuses the calls of one script into kernels and notes that the
// only way to keep data on chip across a global reduction would be persistent
// threads (Section 5, discussion of ATAX and SGEMVT). Here a fixed grid of
// workgroups repeatedly takes the next item from a queue in the workspace and
// processes it with the fused tiles of Algorithm 3 (BiCGK: A read once for
// A p and A^T r) and of the GEMVER plan {ger, ger, gemtv}{gemv}:
//
//   * a whole small instance is one item; for GEMVER the workgroup completes
//     x = beta B^T y + z itself and then runs w = alpha B x, so the global
//     barrier between the two kernels of the plan becomes a workgroup barrier;
//   * a larger instance is cut into row blocks; every block writes a column
//     partial, the last block to arrive (a per-instance counter) adds the
//     partials in block order and, for GEMVER, publishes x with a flag;
//   * the K2 row blocks of split GEMVER instances come after every phase-1
//     item in the queue. A K2 block waits for its flag, which can only be
//     held back by phase-1 items already taken by running workgroups, so the
//     wait always ends; it is bounded all the same and reports an error bit.
//
// Every counter is returned to zero by the item or workgroup that uses it
// last, so the launch can be replayed (e.g. from a graph) without clearing.
//
// Tile shape by size bucket. Up to n = 512: TPR = 2^LTPR lanes share a row (K
// float4 chunks each), 256 / TPR rows are in flight per workgroup step, G =
// 2^LG steps are loaded before their row sums are reduced. Above, BiCGK and
// the first phase of GEMVER let the four waves split the columns of each row
// (below).
#include <hip/hip_runtime.h>

#include "device/kf_blocks.h"
#include "kf_batch_defs.h"

namespace {

// Row sums of G = 2^LG partials per lane over groups of TPR = 2^LTPR lanes:
// a transposing exchange over the top LG bits of the group, then a butterfly
// over the rest. Lane cl of a group returns the sum of row cl >> (LTPR - LG).
template <int LTPR, int LG>
__device__ __forceinline__ float kfb_rows_reduce(float* v) {
    return kf_rows_reduce_from<(1 << LTPR) / 2, (1 << LG)>(v);
}

// a(l) + a(l ^ M) for M = TPR, 2 TPR, ..., 32
template <int M>
__device__ __forceinline__ kf_f4 kfb_fold4(kf_f4 a) {
    if constexpr (M < 64) {
        kf_f4 r;
        r.x = kf_xor_add<M>(a.x); r.y = kf_xor_add<M>(a.y); r.z = kf_xor_add<M>(a.z); r.w = kf_xor_add<M>(a.w);
        return kfb_fold4<2 * M>(r);
    } else {
        return a;
    }
}

// Column sums of acc[k] over the 256 / TPR row-lanes of the workgroup, in a
// fixed order (butterfly inside the wave, then waves 0..3, compensated). emit(c, v) runs in
// threads tid < TPR with chunk c = tid + k TPR (columns 4c .. 4c + 3).
template <int LTPR, int K, typename Emit>
__device__ __forceinline__ void kfb_colsum(kf_f4* acc, kf_f4* red, Emit emit) {
    constexpr int TPR = 1 << LTPR;
    const int lane = __lane_id();
    const int wave = threadIdx.x >> 6;
#pragma unroll
    for (int k = 0; k < K; ++k) acc[k] = kfb_fold4<TPR>(acc[k]);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        __syncthreads();
        if (lane < TPR) red[wave * TPR + lane] = acc[k];
        __syncthreads();
        if (threadIdx.x < TPR) {
            const int t = threadIdx.x;
            kf_cs4 s = kf_cs4_init(red[t]);
            s = kf_cs4_add(s, red[TPR + t]);
            s = kf_cs4_add(s, red[2 * TPR + t]);
            s = kf_cs4_add(s, red[3 * TPR + t]);
            emit(t + k * TPR, kf_cs4_value(s));
        }
    }
}

// Data that another workgroup of the launch reads (column partials, x, and B of a
// split instance) is stored through the XCD's L2 and loaded past it, access by
// access, so publishing it takes a wait for the stores and no fence. A device-scope
// release walks the whole L2 and an acquire empties it for every workgroup of the
// XCD: 512 BiCGK + 512 GEMVER, n = 32 .. 2048, 965 us with fences and 815 without
// (1024 BiCGK alone 454 and 344 us, 5.7 TB/s).
typedef int kfb_i4 __attribute__((ext_vector_type(4)));
constexpr int KFB_STREAM = 2;        // nt
constexpr int KFB_DEV = 16;          // sc1: device scope
constexpr int KFB_DEV_STREAM = 18;   // sc1 nt
__device__ __forceinline__ __amdgpu_buffer_rsrc_t kfb_rsrc(const float* p, long floats) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, (int)(floats * 4), 0x00027000);
}
template <int AUX>
__device__ __forceinline__ kf_f4 kfb_ld4_dev(__amdgpu_buffer_rsrc_t b, int off) {
    return __builtin_bit_cast(kf_f4, __builtin_amdgcn_raw_buffer_load_b128(b, off * 4, 0, AUX));
}
template <int AUX>
__device__ __forceinline__ void kfb_st4_dev(__amdgpu_buffer_rsrc_t b, int off, kf_f4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(kfb_i4, v), b, off * 4, 0, AUX);
}
// at lane offset `off` of the row that starts at the uniform offset `row`
template <int AUX>
__device__ __forceinline__ kf_f4 kfb_ld4_row(__amdgpu_buffer_rsrc_t b, int off, int row) {
    return __builtin_bit_cast(kf_f4, __builtin_amdgcn_raw_buffer_load_b128(b, off * 4, row * 4, AUX));
}
// the first nv (0 .. 4) floats of v
template <int AUX>
__device__ __forceinline__ void kfb_st4_row(__amdgpu_buffer_rsrc_t b, int off, int row, int nv, kf_f4 v) {
    if (nv >= 4) { __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(kfb_i4, v), b, off * 4, row * 4, AUX); return; }
    if (nv > 0) __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v.x), b, off * 4, row * 4, AUX);
    if (nv > 1) __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v.y), b, off * 4 + 4, row * 4, AUX);
    if (nv > 2) __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v.z), b, off * 4 + 8, row * 4, AUX);
}
template <int AUX>
__device__ __forceinline__ void kfb_st4_dev_tail(__amdgpu_buffer_rsrc_t b, int off, int nv, kf_f4 v) {
    if (nv >= 4) { kfb_st4_dev<AUX>(b, off, v); return; }
    if (nv > 0) __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v.x), b, off * 4, 0, KFB_DEV);
    if (nv > 1) __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v.y), b, off * 4 + 4, 0, KFB_DEV);
    if (nv > 2) __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v.z), b, off * 4 + 8, 0, KFB_DEV);
}
// Every store of the workgroup has reached the point that all XCDs share.
__device__ __forceinline__ void kfb_stored() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// Arrival at a per-instance counter. Returns true in every thread of the
// workgroup that arrives last, and the counter is back at zero. Device-scope
// stores made before an arrival are visible to device-scope loads of the last.
__device__ __forceinline__ bool kfb_arrive(unsigned* counter, unsigned count, int* s_flag) {
    kfb_stored();
    if (threadIdx.x == 0) {
        const unsigned old = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int last = old == count - 1;
        if (last) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_flag = last;
    }
    __syncthreads();
    return *s_flag != 0;
}

// Arrival that publishes nothing (only counts): no wait for stores. The K2 blocks of a
// split GEMVER instance use it to find the last one, which clears the
// instance's flag for the next launch; every block has passed its wait on the
// flag before it arrives, and the next launch starts after this one ends.
__device__ __forceinline__ bool kfb_count(unsigned* counter, unsigned count, int* s_flag) {
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned old = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int last = old == count - 1;
        if (last) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_flag = last;
    }
    __syncthreads();
    return *s_flag != 0;
}

// Sixteen loads are in flight: one at a time, each waits for memory past the L2, and
// x of a GEMVER instance for all of them (n = 2048 in 32 blocks: 90 -> 78 us).
constexpr int KFB_AHEAD = 16;
// Sum of the column partials of a split instance's row blocks 0 .. nblk - 1
// (ld floats apart) at columns col .. col + 3, compensated, in
// block order.
__device__ __forceinline__ kf_f4 kfb_block_partials(__amdgpu_buffer_rsrc_t p, int col, int ld, int nblk) {
    kf_cs4 t = kf_cs4_init(kf_zero4());
#pragma unroll 1
    for (int b0 = 0; b0 < nblk; b0 += KFB_AHEAD) {
        kf_f4 v[KFB_AHEAD];
#pragma unroll
        for (int j = 0; j < KFB_AHEAD; ++j) {
            const int b = b0 + j < nblk ? b0 + j : nblk - 1;
            v[j] = kfb_ld4_row<KFB_DEV>(p, col, b * ld);
        }
#pragma unroll
        for (int j = 0; j < KFB_AHEAD; ++j)
            if (b0 + j < nblk) t = kf_cs4_add(t, v[j]);
    }
    return kf_cs4_value(t);
}

// Chunk k of a thread covers columns col .. col + 3, col = 4 (cl + k TPR).
// Per chunk the thread keeps the load column clamped into the row (cc) and
// the number of its columns below n (nv, 0 .. 4), both 32-bit.
struct kfb_cols {
    int cc, nv;
};
__device__ __forceinline__ kfb_cols kfb_col(int col, int n, int ld) {
    kfb_cols c;
    c.cc = col < ld - 4 ? col : ld - 4;
    const int v = n - col;
    c.nv = v < 0 ? 0 : (v > 4 ? 4 : v);
    return c;
}
// Row `row` of a matrix block at one chunk, without branches: the address is
// clamped into the block (row r1 - 1, the row's last chunk) and entries of
// rows >= r1 or columns >= n are replaced by zero with a select (padding may
// hold NaN). Clamped loads fall on lines that other lanes fetch anyway.
__device__ __forceinline__ kf_f4 kfb_mask(kf_f4 v, int row, int r1, kfb_cols c) {
    const int lim = row < r1 ? c.nv : 0;
    v.x = lim > 0 ? v.x : 0.f;
    v.y = lim > 1 ? v.y : 0.f;
    v.z = lim > 2 ? v.z : 0.f;
    v.w = lim > 3 ? v.w : 0.f;
    return v;
}
__device__ __forceinline__ kf_f4 kfb_ldm(const float* M, long ld, int row, int r1, kfb_cols c) {
    const long rc = row < r1 ? row : r1 - 1;
    return kfb_mask(kf_ld4_nt(M + rc * ld + c.cc), row, r1, c);
}
// the same of a matrix that other workgroups have stored
__device__ __forceinline__ kf_f4 kfb_ldm(__amdgpu_buffer_rsrc_t M, int ld, int row, int r1, kfb_cols c) {
    const int rc = row < r1 ? row : r1 - 1;
    return kfb_mask(kfb_ld4_dev<KFB_DEV_STREAM>(M, rc * ld + c.cc), row, r1, c);
}
// Vector entries at one chunk (the vector holds exactly n floats; entries
// at index >= n read as zero). 32-bit index arithmetic throughout.
__device__ __forceinline__ kf_f4 kfb_ldv(const float* v, int col, int n) {
    if (col + 4 <= n) return kf_ld4(v + col);
    kf_f4 r = kf_zero4();
    if (col + 0 < n) r.x = v[col + 0];
    if (col + 1 < n) r.y = v[col + 1];
    if (col + 2 < n) r.z = v[col + 2];
    return r;
}
__device__ __forceinline__ void kfb_stv(float* v, int col, int n, kf_f4 x) {
    if (col + 4 <= n) { kf_st4(v + col, x); return; }
    if (col + 0 < n) v[col + 0] = x.x;
    if (col + 1 < n) v[col + 1] = x.y;
    if (col + 2 < n) v[col + 2] = x.z;
}
__device__ __forceinline__ void kfb_stm(float* row, int col, int n, kf_f4 x) {
    if (col + 4 <= n) { kf_st4_nt(row + col, x); return; }
    if (col + 0 < n) row[col + 0] = x.x;
    if (col + 1 < n) row[col + 1] = x.y;
    if (col + 2 < n) row[col + 2] = x.z;
}

// threadIdx.x as an opaque value: per-thread column offsets are then
// recomputed for every item instead of being hoisted out of the persistent
// loop, where they would stay live across all buckets.
__device__ __forceinline__ int kfb_tid() {
    int t;
    asm volatile("v_mov_b32 %0, %1" : "=v"(t) : "v"((int)threadIdx.x));
    return t;
}

// Column-indexed vectors (BiCGK p; GEMVER v1, v2, then x) are staged in LDS
// once per item and read from there at every row step: held in registers
// they would cost 2 K float4 per lane and halve the occupancy of the
// largest tiles.
// A compiler barrier at the top of each row step: the LDS copies of the
// column vectors are read again at every step instead of being hoisted into
// registers for the whole item.
__device__ __forceinline__ void kfb_reload_lds() { asm volatile("" ::: "memory"); }

struct Shared {
    kf_f4 red[KFB_THREADS];
    kf_f4 cv[2][KFB_MAX_N / 4];
    float rowp[2][4][16];   // wave partials of row sums, double-buffered (wide tiles)
    int flag;
    int item;
};

// Chunks 0 .. TPR K - 1 of a column vector into LDS (threads tid < TPR;
// entries >= n are zero). The caller synchronises before the first read.
template <int LTPR, int K>
__device__ __forceinline__ void kfb_stage(kf_f4* dst, const float* v, int n, int tid) {
    constexpr int TPR = 1 << LTPR;
    if (tid < TPR) {
#pragma unroll
        for (int k = 0; k < K; ++k) dst[tid + k * TPR] = kfb_ldv(v, 4 * (tid + k * TPR), n);
    }
}

// Wait (thread 0, bounded) until the instance's x is published.
// Returns false in every thread if the wait ran out (error bit set).
__device__ __forceinline__ bool kfb_wait_x(unsigned* ctr, unsigned* sync, unsigned spin_limit, Shared& sh) {
    if (threadIdx.x == 0) {
        unsigned spins = 0;
        int ok = 1;
        while (__hip_atomic_load(ctr + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0u) {
            if (++spins > spin_limit) {
                atomicOr(sync + KFB_SYNC_ERROR, KFB_ERR_SPIN);
                ok = 0;
                break;
            }
            __builtin_amdgcn_s_sleep(8);
        }
        sh.flag = ok;
    }
    __syncthreads();
    const bool ready = sh.flag != 0;
    __syncthreads();
    return ready;
}

// w rows r0 .. r1 - 1 of alpha B x, x given per thread at its columns.
template <int LTPR, int K, int LG, typename Mat>
__device__ __forceinline__ void kfb_gemv_rows(const kfb_inst& I, Mat B,
                                              float* __restrict__ w, int r0, int r1, const kf_f4* xv) {
    // xv: x in LDS, chunk c at xv[c]
    constexpr int TPR = 1 << LTPR, G = 1 << LG, RL = KFB_THREADS / TPR, RI = RL * G;
    const int tid = kfb_tid(), cl = tid & (TPR - 1), rl = tid >> LTPR;
    const int n = I.n;
    const int ld = I.ld;
    kfb_cols cs[K];
#pragma unroll
    for (int k = 0; k < K; ++k) cs[k] = kfb_col(4 * (cl + k * TPR), n, I.ld);
#pragma unroll 1
    for (int i0 = r0; i0 < r1; i0 += RI) {
        kfb_reload_lds();
        kf_f4 b[G][K];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int row = i0 + g * RL + rl;
#pragma unroll
            for (int k = 0; k < K; ++k) b[g][k] = kfb_ldm(B, ld, row, r1, cs[k]);
        }
        float wp[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            wp[g] = 0.f;
#pragma unroll
            for (int k = 0; k < K; ++k) wp[g] = kf_dot4(b[g][k], xv[cl + k * TPR], wp[g]);
        }
        const float ws = kfb_rows_reduce<LTPR, LG>(wp);
        const int g = cl >> (LTPR - LG);
        const int row = i0 + g * RL + rl;
        if ((cl & ((TPR >> LG) - 1)) == 0 && row < r1) w[row] = I.alpha * ws;
    }
}

template <int LTPR, int K, int LG>
__device__ void kfb_bicgk(const kfb_inst& I, int blk, float* __restrict__ arena, float* __restrict__ ws,
                          unsigned* sync, Shared& sh) {
    constexpr int TPR = 1 << LTPR, G = 1 << LG, RL = KFB_THREADS / TPR, RI = RL * G;
    const int tid = kfb_tid(), cl = tid & (TPR - 1), rl = tid >> LTPR;
    const int n = I.n;
    const long ld = I.ld;
    const int r0 = blk * I.rows, r1 = min(n, r0 + I.rows);
    const float* __restrict__ A = arena + I.a;
    const float* __restrict__ p = arena + I.v[0];
    const float* __restrict__ r = arena + I.v[1];
    float* __restrict__ q = arena + I.v[2];
    float* __restrict__ s = arena + I.v[3];
    kf_f4 acc[K];
    kfb_cols cs[K];
    kfb_stage<LTPR, K>(sh.cv[0], p, n, tid);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        cs[k] = kfb_col(4 * (cl + k * TPR), n, I.ld);
        acc[k] = kf_zero4();
    }
    __syncthreads();
    const kf_f4* pv = sh.cv[0] + cl;
#pragma unroll 1
    for (int i0 = r0; i0 < r1; i0 += RI) {
        kfb_reload_lds();
        kf_f4 a[G][K];
        float rr[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int row = i0 + g * RL + rl;
            const bool ok = row < r1;
            rr[g] = r[ok ? row : r1 - 1];
            rr[g] = ok ? rr[g] : 0.f;
#pragma unroll
            for (int k = 0; k < K; ++k) a[g][k] = kfb_ldm(A, ld, row, r1, cs[k]);
        }
        float qp[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            qp[g] = 0.f;
#pragma unroll
            for (int k = 0; k < K; ++k) qp[g] = kf_dot4(a[g][k], pv[k * TPR], qp[g]);
#pragma unroll
            for (int k = 0; k < K; ++k) acc[k] = kf_fma4s(rr[g], a[g][k], acc[k]);
        }
        const float qs = kfb_rows_reduce<LTPR, LG>(qp);
        const int g = cl >> (LTPR - LG);
        const int row = i0 + g * RL + rl;
        if ((cl & ((TPR >> LG) - 1)) == 0 && row < r1) q[row] = qs;
    }
    if (I.nblk == 1) {
        kfb_colsum<LTPR, K>(acc, sh.red, [&](int c, kf_f4 v) { kfb_stv(s, 4 * c, n, v); });
        return;
    }
    const __amdgpu_buffer_rsrc_t part = kfb_rsrc(ws + I.ws, (long)I.nblk * I.ld);
    kfb_colsum<LTPR, K>(acc, sh.red, [&](int c, kf_f4 v) {
        if (4 * c < I.ld) kfb_st4_dev<KFB_DEV>(part, blk * I.ld + 4 * c, v);
    });
    unsigned* ctr = sync + KFB_SYNC_HEADER + KFB_SYNC_PER_INST * I.sync;
    if (kfb_arrive(ctr, (unsigned)I.nblk, &sh.flag)) {
        for (int c = threadIdx.x; 4 * c < n; c += KFB_THREADS) {
            kfb_stv(s, 4 * c, n, kfb_block_partials(part, 4 * c, I.ld, I.nblk));
        }
    }
}

// SPLIT: one row block of several (B goes to other workgroups); otherwise the
// whole instance.
template <int LTPR, int K, int LG, bool SPLIT>
__device__ void kfb_gemver_k1(const kfb_inst& I, int blk, float* __restrict__ arena, float* __restrict__ ws,
                              unsigned* sync, Shared& sh) {
    constexpr int TPR = 1 << LTPR, G = 1 << LG, RL = KFB_THREADS / TPR, RI = RL * G;
    const int tid = kfb_tid(), cl = tid & (TPR - 1), rl = tid >> LTPR;
    const int n = I.n;
    const long ld = I.ld;
    const int r0 = blk * I.rows, r1 = min(n, r0 + I.rows);
    const float* __restrict__ A = arena + I.a;
    float* __restrict__ B = arena + I.b;
    const float* __restrict__ u1 = arena + I.v[0];
    const float* __restrict__ v1 = arena + I.v[1];
    const float* __restrict__ u2 = arena + I.v[2];
    const float* __restrict__ v2 = arena + I.v[3];
    const float* __restrict__ y = arena + I.v[4];
    const float* __restrict__ z = arena + I.v[5];
    float* __restrict__ x = arena + I.v[6];
    float* __restrict__ w = arena + I.v[7];
    const __amdgpu_buffer_rsrc_t Bs = kfb_rsrc(B, n * ld);
    (void)Bs;
    kf_f4 acc[K];
    kfb_cols cs[K];
    kfb_stage<LTPR, K>(sh.cv[0], v1, n, tid);
    kfb_stage<LTPR, K>(sh.cv[1], v2, n, tid);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        cs[k] = kfb_col(4 * (cl + k * TPR), n, I.ld);
        acc[k] = kf_zero4();
    }
    __syncthreads();
    const kf_f4* v1c = sh.cv[0] + cl;
    const kf_f4* v2c = sh.cv[1] + cl;
#pragma unroll 1
    for (int i0 = r0; i0 < r1; i0 += RI) {
        kfb_reload_lds();
        kf_f4 a[G][K];
        float u1r[G], u2r[G], yr[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int row = i0 + g * RL + rl;
            const bool ok = row < r1;
            const int rc = ok ? row : r1 - 1;
            u1r[g] = ok ? u1[rc] : 0.f;
            u2r[g] = ok ? u2[rc] : 0.f;
            yr[g] = ok ? y[rc] : 0.f;
#pragma unroll
            for (int k = 0; k < K; ++k) a[g][k] = kfb_ldm(A, ld, row, r1, cs[k]);
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int row = i0 + g * RL + rl;
#pragma unroll
            for (int k = 0; k < K; ++k) {
                kf_f4 b = kf_fma4s(u1r[g], v1c[k * TPR], a[g][k]);
                b = kf_fma4s(u2r[g], v2c[k * TPR], b);
                if constexpr (SPLIT) {
                    if (row < r1) kfb_st4_dev_tail<KFB_DEV_STREAM>(Bs, row * I.ld + 4 * (cl + k * TPR), cs[k].nv, b);
                } else {
                    if (row < r1) kfb_stm(B + (long)row * ld, 4 * (cl + k * TPR), n, b);
                }
                acc[k] = kf_fma4s(yr[g], b, acc[k]);
            }
        }
    }
    if constexpr (!SPLIT) {
        // x is complete inside this workgroup: finish it, then run the gemv.
        kfb_colsum<LTPR, K>(acc, sh.red, [&](int c, kf_f4 v) {
            const kf_f4 xc = kf_fma4s(I.beta, v, kfb_ldv(z, 4 * c, n));
            kfb_stv(x, 4 * c, n, xc);
            sh.cv[0][c] = xc;
        });
        __syncthreads();
        kfb_gemv_rows<LTPR, K, LG>(I, (const float*)B, w, 0, n, sh.cv[0]);
        return;
    }
    const __amdgpu_buffer_rsrc_t part = kfb_rsrc(ws + I.ws, (long)I.nblk * I.ld);
    kfb_colsum<LTPR, K>(acc, sh.red, [&](int c, kf_f4 v) {
        if (4 * c < I.ld) kfb_st4_dev<KFB_DEV>(part, blk * I.ld + 4 * c, v);
    });
    const __amdgpu_buffer_rsrc_t xs = kfb_rsrc(x, n);
    unsigned* ctr = sync + KFB_SYNC_HEADER + KFB_SYNC_PER_INST * I.sync;
    if (kfb_arrive(ctr, (unsigned)I.nblk, &sh.flag)) {
        for (int c = threadIdx.x; 4 * c < n; c += KFB_THREADS) {
            const kf_f4 t = kfb_block_partials(part, 4 * c, I.ld, I.nblk);
            kfb_st4_dev_tail<KFB_DEV>(xs, 4 * c, n - 4 * c, kf_fma4s(I.beta, t, kfb_ldv(z, 4 * c, n)));
        }
        kfb_stored();
        if (threadIdx.x == 0) __hip_atomic_store(ctr + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---- wide BiCGK tiles (n > 512): the four waves split each row's columns ---
// Lane t of the workgroup owns chunks t + 256 k (k < K) of every row of the
// item, so the column result A^T r needs no cross-lane reduction; G rows
// are loaded per step, and a row sum is finished by a transposing reduction
// inside each wave and then the four wave partials, added in wave order after
// one barrier per step (double-buffered in LDS). This is the row-resident
// layout of the single-instance kernels at batch-instance size; it keeps the
// per-lane state small, so more waves are resident.

// Row-indexed scalars of the wide tiles: lanes 0 .. G - 1 load v[i0 + lane]
// (zero past r1) one step ahead; kfb_row_bcast reads each lane as a
// wave-uniform value once the load has long completed.
template <int G>
__device__ __forceinline__ float kfb_row_fetch(const float* v, int i0, int r1) {
    const int lane = __lane_id();
    return (lane < G && i0 + lane < r1) ? v[i0 + lane] : 0.f;
}
template <int G>
__device__ __forceinline__ void kfb_row_bcast(float x, float* out) {
#pragma unroll
    for (int g = 0; g < G; ++g) out[g] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), g));
}

template <int K, int LG>
__device__ __forceinline__ void kfb_w_rows_sum(const float* qp_in, float* __restrict__ out, float scale, int i0,
                                               int r1, Shared& sh, int& buf) {
    constexpr int G = 1 << LG;
    float qp[G];
#pragma unroll
    for (int g = 0; g < G; ++g) qp[g] = qp_in[g];
    const float sw = kfb_rows_reduce<6, LG>(qp);
    const int lane = __lane_id(), wave = threadIdx.x >> 6;
    if ((lane & ((64 >> LG) - 1)) == 0) sh.rowp[buf][wave][lane >> (6 - LG)] = sw;
    __syncthreads();
    if (threadIdx.x < G && i0 + (int)threadIdx.x < r1) {
        const int g = threadIdx.x;
        kf_cs t = kf_cs_init(sh.rowp[buf][0][g]);
        t = kf_cs_add(t, sh.rowp[buf][1][g]);
        t = kf_cs_add(t, sh.rowp[buf][2][g]);
        t = kf_cs_add(t, sh.rowp[buf][3][g]);
        out[i0 + g] = scale * kf_cs_value(t);
    }
    buf ^= 1;
}

template <int K, int LG>
__device__ void kfb_w_bicgk(const kfb_inst& I, int blk, float* __restrict__ arena, float* __restrict__ ws,
                            unsigned* sync, Shared& sh) {
    constexpr int G = 1 << LG;
    const int t = kfb_tid();
    const int n = I.n;
    const long ld = I.ld;
    const int r0 = blk * I.rows, r1 = min(n, r0 + I.rows);
    const float* __restrict__ A = arena + I.a;
    const float* __restrict__ r = arena + I.v[1];
    float* __restrict__ q = arena + I.v[2];
    float* __restrict__ s = arena + I.v[3];
    kf_f4 pv[K], acc[K];
    kfb_cols cs[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        cs[k] = kfb_col(4 * (t + 256 * k), n, I.ld);
        pv[k] = kfb_ldv(arena + I.v[0], 4 * (t + 256 * k), n);
        acc[k] = kf_zero4();
    }
    int buf = 0;
    float r_next = kfb_row_fetch<G>(r, r0, r1);
#pragma unroll 1
    for (int i0 = r0; i0 < r1; i0 += G) {
        const float r_cur = r_next;
        kf_f4 a[G][K];
        float rr[G];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int k = 0; k < K; ++k) a[g][k] = kfb_ldm(A, ld, i0 + g, r1, cs[k]);
        r_next = kfb_row_fetch<G>(r, i0 + G, r1);     // issued after this step's matrix loads
        kfb_row_bcast<G>(r_cur, rr);
        float qp[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            qp[g] = 0.f;
#pragma unroll
            for (int k = 0; k < K; ++k) qp[g] = kf_dot4(a[g][k], pv[k], qp[g]);
#pragma unroll
            for (int k = 0; k < K; ++k) acc[k] = kf_fma4s(rr[g], a[g][k], acc[k]);
        }
        kfb_w_rows_sum<K, LG>(qp, q, 1.f, i0, r1, sh, buf);
    }
    if (I.nblk == 1) {
#pragma unroll
        for (int k = 0; k < K; ++k) kfb_stv(s, 4 * (t + 256 * k), n, acc[k]);
        return;
    }
    const __amdgpu_buffer_rsrc_t part = kfb_rsrc(ws + I.ws, (long)I.nblk * I.ld);
#pragma unroll
    for (int k = 0; k < K; ++k)
        if (4 * (t + 256 * k) < I.ld) kfb_st4_dev<KFB_DEV>(part, blk * I.ld + 4 * (t + 256 * k), acc[k]);
    unsigned* ctr = sync + KFB_SYNC_HEADER + KFB_SYNC_PER_INST * I.sync;
    if (kfb_arrive(ctr, (unsigned)I.nblk, &sh.flag)) {
        for (int c = threadIdx.x; 4 * c < n; c += KFB_THREADS) {
            kfb_stv(s, 4 * c, n, kfb_block_partials(part, 4 * c, I.ld, I.nblk));
        }
    }
}

// ---- GEMVER with whole waves per row (n > 128) --------------------------------
// Rows are wave-uniform, so an address is a scalar row offset plus one lane
// register per chunk, and the next step's loads are issued before this step's
// stores of B: loads and stores retire in one order, and a wait for loads behind
// device-scope stores would be a wait for those too. Bound by HBM (A read, B
// written, B read again): 512 BiCGK + 512 GEMVER 815 -> 780 us, 300 + 300 of n =
// 600 .. 1000 673 -> 584; few instances by the latency of a step: 8 GEMVER of n =
// 1000 131 -> 74 us.

// w rows r0 .. r1 - 1 of alpha B x, a wave per row, x in LDS (zero past n).
template <int K, int LG, int AUX>
__device__ __forceinline__ void kfb_w_gemv(const kfb_inst& I, __amdgpu_buffer_rsrc_t B, float* __restrict__ w, int r0,
                                           int r1, const kf_f4* xv) {
    constexpr int G = 1 << LG;
    const int t = kfb_tid(), lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int n = I.n, ld = I.ld;
    kfb_cols cs[K];
#pragma unroll
    for (int k = 0; k < K; ++k) cs[k] = kfb_col(4 * (lane + 64 * k), n, ld);
    kf_f4 bn[G][K];
    auto load = [&](int base) {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int rc = base + g < r1 ? base + g : r1 - 1;
#pragma unroll
            for (int k = 0; k < K; ++k) bn[g][k] = kfb_ld4_row<AUX>(B, cs[k].cc, rc * ld);
        }
    };
    int i = r0 + wave * G;
    load(i);
#pragma unroll 1
    for (; i < r1; i += 4 * G) {
        kfb_reload_lds();
        kf_f4 b[G][K];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int k = 0; k < K; ++k) b[g][k] = kfb_mask(bn[g][k], 0, 1, cs[k]);
        if (i + 4 * G < r1) load(i + 4 * G);
        float wp[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            wp[g] = 0.f;
#pragma unroll
            for (int k = 0; k < K; ++k) wp[g] = kf_dot4(b[g][k], xv[lane + 64 * k], wp[g]);
        }
        const float s = kfb_rows_reduce<6, LG>(wp);
        const int row = i + (lane >> (6 - LG));
        if ((lane & ((64 >> LG) - 1)) == 0 && row < r1) w[row] = I.alpha * s;
    }
}

// K1: WC waves share a row (4 above n = 512: lane t of the workgroup owns chunks
// t + 256 k of every row and its column sums need no exchange; 1 below: four row
// groups whose column sums meet in LDS). A step's G rows are summed first, and where
// one lane has all rows of a block the steps' sums meet as pairs, as those of four
// row groups did: no longer FP32 chains than theirs.
template <int WC, int K, int LG, bool SPLIT>
__device__ void kfb_w_gemver_k1(const kfb_inst& I, int blk, float* __restrict__ arena, float* __restrict__ ws,
                                unsigned* sync, Shared& sh) {
    constexpr int G = 1 << LG, CT = 64 * WC, RW = 4 / WC * G, AUX = SPLIT ? KFB_DEV_STREAM : KFB_STREAM;
    const int t = kfb_tid(), wave = __builtin_amdgcn_readfirstlane(t >> 6), ct = t & (CT - 1);
    const int n = I.n, ld = I.ld;
    const int r0 = blk * I.rows, r1 = min(n, r0 + I.rows);
    const __amdgpu_buffer_rsrc_t A = kfb_rsrc(arena + I.a, n * ld), B = kfb_rsrc(arena + I.b, n * ld);
    const float* __restrict__ u1 = arena + I.v[0];
    const float* __restrict__ u2 = arena + I.v[2];
    const float* __restrict__ y = arena + I.v[4];
    const float* __restrict__ z = arena + I.v[5];
    float* __restrict__ x = arena + I.v[6];
    kf_f4 v1[K], v2[K], acc[K];
    kf_cs4 tot[K];   // WC 4: a lane has all rows of the block, its steps' sums meet as pairs
    kfb_cols cs[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int col = 4 * (ct + CT * k);
        cs[k] = kfb_col(col, n, ld);
        v1[k] = kfb_ldv(arena + I.v[1], col, n);
        v2[k] = kfb_ldv(arena + I.v[3], col, n);
        acc[k] = kf_zero4();
        tot[k] = kf_cs4_init(kf_zero4());
    }
    kf_f4 an[G][K];
    float u1n, u2n, yn;
    auto load = [&](int base) {
        u1n = kfb_row_fetch<G>(u1, base, r1);
        u2n = kfb_row_fetch<G>(u2, base, r1);
        yn = kfb_row_fetch<G>(y, base, r1);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int rc = base + g < r1 ? base + g : r1 - 1;
#pragma unroll
            for (int k = 0; k < K; ++k) an[g][k] = kfb_ld4_row<KFB_STREAM>(A, cs[k].cc, rc * ld);
        }
    };
    int i = r0 + (WC == 4 ? 0 : wave * G);
    load(i);
#pragma unroll 1
    for (; i < r1; i += RW) {
        float u1r[G], u2r[G], yr[G];
        kfb_row_bcast<G>(u1n, u1r);
        kfb_row_bcast<G>(u2n, u2r);
        kfb_row_bcast<G>(yn, yr);
        kf_f4 b[G][K], s[K];
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int k = 0; k < K; ++k) b[g][k] = kf_fma4s(u2r[g], v2[k], kf_fma4s(u1r[g], v1[k], an[g][k]));
        if (i + RW < r1) load(i + RW);
#pragma unroll
        for (int k = 0; k < K; ++k) s[k] = kf_mul4s(yr[0], b[0][k]);
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (i + g < r1) {
#pragma unroll
                for (int k = 0; k < K; ++k) {
                    if (g > 0) s[k] = kf_fma4s(yr[g], b[g][k], s[k]);
                    kfb_st4_row<AUX>(B, 4 * (ct + CT * k), (i + g) * ld, cs[k].nv, b[g][k]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if constexpr (WC == 4) tot[k] = kf_cs4_add(tot[k], s[k]);
            else acc[k] += s[k];
        }
    }
    // column sums of the block at chunk c, each chunk from one thread
    auto columns = [&](auto emit) {
        if constexpr (WC == 4) {
#pragma unroll
            for (int k = 0; k < K; ++k) emit(t + 256 * k, kf_cs4_value(tot[k]));
        } else {
            kfb_colsum<6, K>(acc, sh.red, emit);
        }
    };
    const __amdgpu_buffer_rsrc_t xs = kfb_rsrc(x, n);
    if constexpr (!SPLIT) {
        // x is complete inside this workgroup: finish it, then run the gemv.
        columns([&](int c, kf_f4 v) {
            const kf_f4 xc = 4 * c < n ? kf_fma4s(I.beta, v, kfb_ldv(z, 4 * c, n)) : kf_zero4();
            kfb_stv(x, 4 * c, n, xc);
            sh.cv[0][c] = kfb_mask(xc, 0, 1, kfb_col(4 * c, n, ld));
        });
        __syncthreads();
        kfb_w_gemv<K * WC, (WC == 4 ? LG - 2 : LG), KFB_STREAM>(I, B, arena + I.v[7], 0, n, sh.cv[0]);
        return;
    }
    const __amdgpu_buffer_rsrc_t part = kfb_rsrc(ws + I.ws, (long)I.nblk * ld);
    columns([&](int c, kf_f4 v) {
        if (4 * c < ld) kfb_st4_dev<KFB_DEV>(part, blk * ld + 4 * c, v);
    });
    unsigned* ctr = sync + KFB_SYNC_HEADER + KFB_SYNC_PER_INST * I.sync;
    if (kfb_arrive(ctr, (unsigned)I.nblk, &sh.flag)) {
        for (int c = threadIdx.x; 4 * c < n; c += KFB_THREADS) {
            const kf_f4 v = kfb_block_partials(part, 4 * c, ld, I.nblk);
            kfb_st4_dev_tail<KFB_DEV>(xs, 4 * c, n - 4 * c, kf_fma4s(I.beta, v, kfb_ldv(z, 4 * c, n)));
        }
        kfb_stored();
        if (threadIdx.x == 0) __hip_atomic_store(ctr + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// K2 block of a split instance: CHUNKS float4 cover x; gemv(B, r0, r1) walks the
// block's rows.
template <int CHUNKS, typename Gemv>
__device__ __forceinline__ void kfb_gemver_k2(const kfb_inst& I, int blk, float* __restrict__ arena, unsigned* sync,
                                              unsigned spin_limit, Shared& sh, Gemv gemv) {
    const int n = I.n;
    unsigned* ctr = sync + KFB_SYNC_HEADER + KFB_SYNC_PER_INST * I.sync;
    if (!kfb_wait_x(ctr, sync, spin_limit, sh)) return;
    // (a vector's place in the arena is a multiple of 64 floats)
    const __amdgpu_buffer_rsrc_t x = kfb_rsrc(arena + I.v[6], (n + 3) / 4 * 4);
    for (int c = threadIdx.x; c < CHUNKS; c += KFB_THREADS) {
        const kfb_cols cx = kfb_col(4 * c, n, (n + 3) / 4 * 4);
        sh.cv[0][c] = kfb_mask(kfb_ld4_dev<KFB_DEV>(x, cx.cc), 0, 1, cx);
    }
    __syncthreads();
    const int r0 = blk * I.rows, r1 = min(n, r0 + I.rows);
    gemv(kfb_rsrc(arena + I.b, n * I.ld), r0, r1);
    // the last K2 block of the instance clears the flag for the next launch
    if (kfb_count(ctr + 2, (unsigned)I.nblk, &sh.flag) && threadIdx.x == 0)
        __hip_atomic_store(ctr + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Tile T of the menu of (KIND, B), instantiated from the shared table.
template <int KIND, int B, int T>
__device__ __forceinline__ void kfb_tile_run(const kfb_inst& I, int phase, int blk, float* arena, float* ws,
                                             unsigned* sync, unsigned spin_limit, Shared& sh) {
    constexpr kfb_tile x = kfb_tile_menu[KIND][B][T];
    if constexpr (x.k == 0) {
        return;   // not on the menu (the host never selects it)
    } else if constexpr (KIND == 0 && x.wide) {
        kfb_w_bicgk<x.k, x.lg>(I, blk, arena, ws, sync, sh);
    } else if constexpr (KIND == 0) {
        kfb_bicgk<x.ltpr, x.k, x.lg>(I, blk, arena, ws, sync, sh);
    } else if constexpr (x.ltpr == 6) {
        // whole waves per row; from four chunks a lane on, K1's waves share the rows
        // of a step instead of taking them in turn (the same rows per step)
        constexpr int WC = x.k >= 4 ? 4 : 1, K = x.k / WC, LG = WC == 4 ? x.lg + 2 : x.lg;
        if (phase == KFB_GEMVER_K1) {
            if (I.nblk == 1) kfb_w_gemver_k1<WC, K, LG, false>(I, blk, arena, ws, sync, sh);
            else kfb_w_gemver_k1<WC, K, LG, true>(I, blk, arena, ws, sync, sh);
        } else {
            kfb_gemver_k2<64 * x.k>(I, blk, arena, sync, spin_limit, sh, [&](__amdgpu_buffer_rsrc_t Bm, int r0, int r1) {
                kfb_w_gemv<x.k, x.lg, KFB_DEV_STREAM>(I, Bm, arena + I.v[7], r0, r1, sh.cv[0]);
            });
        }
    } else if (phase == KFB_GEMVER_K1) {
        if (I.nblk == 1) kfb_gemver_k1<x.ltpr, x.k, x.lg, false>(I, blk, arena, ws, sync, sh);
        else kfb_gemver_k1<x.ltpr, x.k, x.lg, true>(I, blk, arena, ws, sync, sh);
    } else {
        kfb_gemver_k2<(x.k << x.ltpr)>(I, blk, arena, sync, spin_limit, sh, [&](__amdgpu_buffer_rsrc_t Bm, int r0, int r1) {
            kfb_gemv_rows<x.ltpr, x.k, x.lg>(I, Bm, arena + I.v[7], r0, r1, sh.cv[0]);
        });
    }
}

template <int KIND, int B, bool MENU>
__device__ __forceinline__ void kfb_bucket_run(const kfb_inst& I, int phase, int blk, float* arena, float* ws,
                                               unsigned* sync, unsigned spin_limit, Shared& sh) {
    if constexpr (MENU) {
        if (I.tile == 1) { kfb_tile_run<KIND, B, 1>(I, phase, blk, arena, ws, sync, spin_limit, sh); return; }
        if (I.tile == 2) { kfb_tile_run<KIND, B, 2>(I, phase, blk, arena, ws, sync, spin_limit, sh); return; }
    }
    kfb_tile_run<KIND, B, 0>(I, phase, blk, arena, ws, sync, spin_limit, sh);
}

template <int KIND, bool MENU>
__device__ __forceinline__ void kfb_kind_run(const kfb_inst& I, int phase, int blk, float* arena, float* ws,
                                             unsigned* sync, unsigned spin_limit, Shared& sh) {
    switch (I.bucket) {
    case 0: kfb_bucket_run<KIND, 0, MENU>(I, phase, blk, arena, ws, sync, spin_limit, sh); break;
    case 1: kfb_bucket_run<KIND, 1, MENU>(I, phase, blk, arena, ws, sync, spin_limit, sh); break;
    case 2: kfb_bucket_run<KIND, 2, MENU>(I, phase, blk, arena, ws, sync, spin_limit, sh); break;
    case 3: kfb_bucket_run<KIND, 3, MENU>(I, phase, blk, arena, ws, sync, spin_limit, sh); break;
    case 4: kfb_bucket_run<KIND, 4, MENU>(I, phase, blk, arena, ws, sync, spin_limit, sh); break;
    default: kfb_bucket_run<KIND, 5, MENU>(I, phase, blk, arena, ws, sync, spin_limit, sh); break;
    }
}

// Three waves per SIMD (168 VGPRs): GEMVER's steps of eight 16-byte loads per lane
// keep the next step's loads beside them.
// MENU: with every tile of the menu, for batches that ask for one that is not the
// default. Without them the code is a third of the size; its first pass through each
// CU's instruction cache is what a few small instances wait for (64 GEMVER of n = 128:
// 27.9 us without the menu, 32.2 with it; 512 of them 39.6 and 43.8).
template <bool MENU>
__global__ void __launch_bounds__(KFB_THREADS) __attribute__((amdgpu_waves_per_eu(3, 8)))
kfb_kernel(const kfb_inst* __restrict__ insts, const kfb_item* __restrict__ items, int nitems, int item0,
           int persistent, float* arena, float* ws, unsigned* sync, unsigned spin_limit) {
    __shared__ Shared sh;
    for (;;) {
        int it;
        if (persistent) {
            if (threadIdx.x == 0) sh.item = (int)atomicAdd(sync + KFB_SYNC_QUEUE, 1u);
            __syncthreads();
            it = sh.item;
            __syncthreads();
            if (it >= nitems) break;
        } else {
            it = item0 + (int)blockIdx.x;
        }
        const kfb_item item = items[it];
        const kfb_inst I = insts[item.inst];
        const int phase = item.phase_blk >> 24;
        const int blk = item.phase_blk & 0xffffff;
        // the instance's tile from the menu of its kind and size bucket
        if (I.kind == 0) kfb_kind_run<0, MENU>(I, phase, blk, arena, ws, sync, spin_limit, sh);   // BiCGK
        else kfb_kind_run<1, MENU>(I, phase, blk, arena, ws, sync, spin_limit, sh);
        if (!persistent) break;
        __syncthreads();
    }
    if (persistent && threadIdx.x == 0) {
        if (atomicAdd(sync + KFB_SYNC_EXIT, 1u) == gridDim.x - 1) {
            __hip_atomic_store(sync + KFB_SYNC_QUEUE, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(sync + KFB_SYNC_EXIT, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

}  // namespace

// Persistent launch (grid workgroups draining the queue) or a direct launch of
// items item0 .. item0 + grid - 1, one per workgroup.
hipError_t kfb_launch(bool menu, const kfb_inst* insts, const kfb_item* items, int nitems, int item0, int grid,
                      int persistent, float* arena, float* ws, unsigned* sync, unsigned spin_limit, hipStream_t st) {
    if (grid <= 0) return hipSuccess;
    hipLaunchKernelGGL(menu ? kfb_kernel<true> : kfb_kernel<false>, dim3(grid), dim3(KFB_THREADS), 0, st, insts, items, nitems, item0, persistent,
                       arena, ws, sync, spin_limit);
    return hipGetLastError();
}

hipError_t kfb_resident_blocks(bool menu, int* per_cu, int* cus) {
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, menu ? kfb_kernel<true> : kfb_kernel<false>, KFB_THREADS, 0);
    if (e != hipSuccess) return e;
    int dev = 0;
    e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    return hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev);
}

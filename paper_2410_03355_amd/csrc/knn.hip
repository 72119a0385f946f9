// Codebook neighbour table B_k (Section 4.2; Algorithm 2, precompute part).
//
// Pipeline per block of query rows:
//   1. approximate keys (fp32) for every pair (query i, token j) into the
//      workspace: squared l2 distance, or minus cosine similarity
//   2. per row: find a threshold with at least k-1+pad approximate keys at or below it
//      (a histogram of the row's list, or bisection with counting passes over a whole row), recompute
//      the survivors' keys in fp64 exactly as the definition states (coordinate
//      order, every operation rounded separately), rank them by (key, index) (buckets over the
//      keys' range; a sorting network for more than 1024 of them or for many equal keys)
//      and emit the first k-1 after the token itself.  A row is emitted only if
//      the approximation's error bound proves no discarded token could belong
//      to it; otherwise it is flagged.
//   3. flagged rows: fp64 keys for all V tokens and ranking by counting.
// The written order is therefore always the fp64 one.
//
// Vocabularies of 4096 tokens and more (aligned codebooks, k from about 60 to about 1000) never form the
// whole key block: a row's threshold is first estimated from the keys to a stratified sample of
// one token in eight, the contraction then runs with an epilogue that appends only the
// (key, token) pairs at or below the row's threshold to a short per-row list, and step 2 works
// on that list.  The threshold only decides how many candidates a row gets; the proof condition
// of step 2 is unchanged (every token left out has an approximate key above every key kept),
// and a row whose list came out too short or too long is flagged like any other.
#include <hip/hip_runtime.h>
#include <limits.h>
#include <math.h>
#include <stdint.h>

#include <mutex>

#include "device_utils.h"
#include "knn_args.h"
#include "knn_plan.h"
#include "lantern.h"
#include "lds_sort.h"

namespace lantern {

// Query rows per pass through the workspace: as many as give a key block of at most 512 MiB, up to
// 8192 (few, full launches: V = 8192 in one block measured 0.44 ms against 0.53 ms in four).
constexpr int ROW_BLOCK = 8192;
static int whole_row_block(int V) {
    const int64_t fit = ((int64_t)512 << 20) / (4 * (int64_t)V) / 128 * 128;
    return fit >= ROW_BLOCK ? ROW_BLOCK : (fit < 128 ? 128 : (int)fit);
}
// The same on the path that keeps candidate lists instead of whole rows: the lists are short, so a
// 16384-token vocabulary goes through in one block (measured at 2048 / 4096 / 8192 / 16384 rows per
// block: 1.10 / 0.93 / 0.82 / 0.77 ms for V = 16384, k = 1000; fewer, fuller launches).
constexpr int FILTER_ROW_BLOCK = 16384;
constexpr int CAND_CAP = 4096;    // candidate slots per row held in LDS
constexpr int SLOW_WGS = 128;     // workgroups (and fp64 row buffers) of the exact pass

__host__ __device__ inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// The sampled-threshold path reads its operands from copies in the order in which the matrix cores
// take them: 32 tokens to a tile, and per tile and step (16 bf16 or 8 fp32 coordinates) the 16 bytes of
// each of the 64 lanes one after the other, so that an operand is one contiguous load of 1 KiB (read from the
// codebook itself a load touches 32 rows, each a cache line of its own).
constexpr size_t PACKED_STEP_BYTES = 64 * 16;
__host__ __device__ inline size_t packed_tiles(int tokens) { return ((size_t)tokens + 31) / 32; }
__host__ __device__ inline size_t packed_steps(int d, int cb_dtype) { return cb_dtype == 1 ? ((size_t)d + 15) / 16 : ((size_t)d + 7) / 8; }

// Largest sample whose keys to 32 rows fit the registers of one workgroup (knn_thresholds).
constexpr int THRESHOLDS_MAX_S = 2048;

struct KnnLayout {
    size_t stats, norms, nmax, dist, flags, slow, total;
    // sampled-threshold path (filter.use): the codebook and the sample as matrix-core operands, what the
    // contraction folds in per token and per sampled token, the sample's norms and a row block's keys to it (samples
    // too large for knn_thresholds only), its thresholds, list lengths and candidate lists; `dist` is then not laid out
    size_t packed, spacked, fold, sfold, snorms, skeys, thr, counts, cand;
    FilterPlan filter;
    int row_block;   // query rows per pass through the key block
    int slow_wgs;    // workgroups (and fp64 row buffers) of the exact pass
};

static KnnLayout knn_layout(int V, int d, int cb_dtype, const FilterPlan& plan, int row_block, int slow_wgs) {
    KnnLayout L;
    L.filter = plan;
    L.row_block = V < row_block ? V : row_block;
    L.slow_wgs = slow_wgs;
    size_t off = 0;
    L.stats = off; off = align_up(off + 256, 256);   // int32[0]: rows that took the exact all-pairs pass
    L.norms = off; off = align_up(off + sizeof(float) * (size_t)V, 256);
    L.nmax = off;  off = align_up(off + 256, 256);
    L.dist = L.packed = L.spacked = L.fold = L.sfold = L.snorms = L.skeys = L.thr = L.counts = L.cand = off;
    if (plan.use) {
        const size_t steps = packed_steps(d, cb_dtype);
        L.packed = off;  off = align_up(off + packed_tiles(V) * steps * PACKED_STEP_BYTES, 256);
        L.spacked = off; off = align_up(off + packed_tiles(plan.S) * steps * PACKED_STEP_BYTES, 256);
        L.fold = off;    off = align_up(off + sizeof(float) * 32 * packed_tiles(V), 256);
        L.sfold = off;   off = align_up(off + sizeof(float) * (size_t)plan.S, 256);
        L.snorms = off; off = align_up(off + sizeof(float) * (size_t)plan.S, 256);
        L.skeys = off;
        if (plan.S > THRESHOLDS_MAX_S) off = align_up(off + sizeof(float) * (size_t)L.row_block * plan.S, 256);
        L.thr = off;    off = align_up(off + sizeof(float) * (size_t)L.row_block, 256);
        L.counts = off; off = align_up(off + sizeof(int) * (size_t)L.row_block, 256);
        L.cand = off;   off = align_up(off + (plan.tokens ? sizeof(uint32_t) : sizeof(uint2)) * (size_t)L.row_block * plan.cap, 256);
    } else {
        L.dist = off;   off = align_up(off + sizeof(float) * (size_t)L.row_block * V, 256);
    }
    L.flags = off; off = align_up(off + sizeof(int) * (size_t)V, 256);   // one word per row of the table
    L.slow = off;  off = align_up(off + sizeof(double) * (size_t)L.slow_wgs * V, 256);
    L.total = off;
    return L;
}

// The largest layout of the given path that fits `bytes`: as many query rows per pass as the
// rest holds (a multiple of 128, the contraction's tile).  row_block 0: nothing fits.
static KnnLayout knn_layout_within(int V, int d, int cb_dtype, const FilterPlan& plan, int slow_wgs, size_t bytes) {
    for (int rb = whole_row_block(V); rb >= 128; rb -= 128) {
        const KnnLayout L = knn_layout(V, d, cb_dtype, plan, rb, slow_wgs);
        if (L.total <= bytes) return L;
    }
    KnnLayout none = knn_layout(V, d, cb_dtype, plan, 128, slow_wgs);
    none.row_block = 0;
    return none;
}

static const FilterPlan NO_FILTER = {false, false, false, 0, 0, 0, 0};

// What lantern_build_knn asks of its caller: the layout of the path the shape takes, and where that one filters at least
// that of whole key blocks: a codebook that turns out not to be 16-byte aligned falls back to those,
// and fewer rows to a pass leave part of the device idle in its selection (the size of the lists alone / this one:
// V = 16384 bf16, k = 100, 960 / 8192 rows 2594 / 2357 us; V = 33000, k = 230, 2900 / 3968 rows 21.9 / 19.6 ms).
size_t knn_workspace_bytes(int V, int d, int k, int cb_dtype) {
    const FilterPlan plan = filter_plan(V, d, k, cb_dtype);
    const size_t whole = knn_layout(V, d, cb_dtype, NO_FILTER, whole_row_block(V), SLOW_WGS).total;
    if (!plan.use) return whole;
    const size_t lists = knn_layout(V, d, cb_dtype, plan, FILTER_ROW_BLOCK, SLOW_WGS).total;
    return lists > whole ? lists : whole;
}

// ---- scratch of the entry point that allocates nothing ----
// Device memory that lives as long as the process, one copy per GPU.  Host code never uses the
// array's name as an address: it asks the runtime for the array's device address once per device
// and passes that pointer on.
constexpr size_t STATIC_SCRATCH_BYTES = LANTERN_STATIC_SCRATCH_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_SCRATCH_BYTES];

// The static scratch serves the whole-key-block path with fewer exact-pass buffers and as many
// query rows per pass as fit.  row_block 0: V is beyond what the scratch can serve.
constexpr int STATIC_SLOW_WGS = 32;
static KnnLayout knn_layout_static(int V, int d, int cb_dtype) {
    return knn_layout_within(V, d, cb_dtype, NO_FILTER, STATIC_SLOW_WGS, STATIC_SCRATCH_BYTES);
}

bool knn_static_fits(int V) { return knn_layout_static(V, 4, 0).row_block > 0; }

// Device address of the static scratch on the current device (looked up once per device).
static hipError_t static_scratch_ptr(void** out) {
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static void* ptrs[MAX_DEVICES];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptrs[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        ptrs[dev] = p;
    }
    *out = ptrs[dev];
    return hipSuccess;
}

template <typename CT> __device__ __forceinline__ float cb_f32(const CT* p, int64_t i);
template <> __device__ __forceinline__ float cb_f32<float>(const float* p, int64_t i) { return p[i]; }
template <> __device__ __forceinline__ float cb_f32<uint16_t>(const uint16_t* p, int64_t i) {
    return __uint_as_float(static_cast<uint32_t>(p[i]) << 16);
}

// order-preserving map float -> uint32 (ascending)
__device__ __forceinline__ uint32_t ord_key(float f) {
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float ord_inv(uint32_t k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// ---- exact fp64 key of the pair (i, j): the definition, operation by operation ----
// Four consecutive coordinates of a code as floats (one 16-byte or 8-byte load); the caller
// guarantees t + 3 < d and 16-byte aligned rows.
__device__ __forceinline__ void cb_load4(const float* p, int t, float (&o)[4]) {
    const float4 v = *reinterpret_cast<const float4*>(p + t);
    o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w;
}
__device__ __forceinline__ void cb_load4(const uint16_t* p, int t, float (&o)[4]) {
    const uint2 v = *reinterpret_cast<const uint2*>(p + t);
    o[0] = __uint_as_float(v.x << 16); o[1] = __uint_as_float(v.x & 0xFFFF0000u);
    o[2] = __uint_as_float(v.y << 16); o[3] = __uint_as_float(v.y & 0xFFFF0000u);
}

// vec4: rows are 16-byte aligned and d is a multiple of 4, so coordinates are fetched four at
// a time; the arithmetic is the same sequence of separately rounded operations either way.
template <typename CT>
__device__ double exact_key(const CT* cb, int d, int i, int j, int metric, bool vec4) {
#pragma clang fp contract(off)
    const CT* ci = cb + (int64_t)i * d;
    const CT* cj = cb + (int64_t)j * d;
    if (metric == 0) {
        double acc = 0.0;
        if (vec4) {
#pragma unroll 4   // the loads of four groups are in flight together; the sum keeps its order
            for (int t = 0; t < d; t += 4) {
                float x[4], y[4];
                cb_load4(ci, t, x);
                cb_load4(cj, t, y);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double diff = (double)x[e] - (double)y[e];
                    const double sq = diff * diff;
                    acc = acc + sq;
                }
            }
        } else {
            for (int t = 0; t < d; ++t) {
                const double diff = (double)cb_f32<CT>(ci, t) - (double)cb_f32<CT>(cj, t);
                const double sq = diff * diff;
                acc = acc + sq;
            }
        }
        return acc == acc ? acc : (double)INFINITY;
    }
    double ni = 0.0, nj = 0.0, dot = 0.0;
    for (int t = 0; t < d; ++t) {
        const double x = (double)cb_f32<CT>(ci, t);
        const double y = (double)cb_f32<CT>(cj, t);
        const double xx = x * x;
        const double yy = y * y;
        const double xy = x * y;
        ni = ni + xx;
        nj = nj + yy;
        dot = dot + xy;
    }
    ni = sqrt(ni);
    nj = sqrt(nj);
    const double den = ni * nj;
    const double key = -(dot / den);
    return key == key ? key : (double)INFINITY;   // no similarity (a code of zero norm): the farthest
}

// The same key for rows of whole 16-byte vectors at aligned addresses, the row's own code as doubles in LDS (`own`).
// The arithmetic is the definition's, in its order; U vectors of the other code are on their way together.
// norm2 (cosine key): the sum of squares of the row's own code, in order.
typedef uint32_t vec4u __attribute__((ext_vector_type(4)));
template <typename CT, int METRIC>
struct KeySum {
    static constexpr int EPV = 16 / (int)sizeof(CT);
    double acc = 0.0, nj = 0.0;
    __device__ __forceinline__ void add(const vec4u& v, const double* own) {
#pragma clang fp contract(off)
#pragma unroll
        for (int e = 0; e < EPV; ++e) {
            const uint32_t word = EPV == 4 ? v[e] : v[e >> 1];
            const float yf = EPV == 4 ? __uint_as_float(word) : __uint_as_float((e & 1) ? (word & 0xFFFF0000u) : (word << 16));
            const double x = own[e], y = (double)yf;
            if (METRIC == 0) {
                const double diff = x - y;
                const double sq = diff * diff;
                acc = acc + sq;
            } else {
                const double yy = y * y;
                const double xy = x * y;
                nj = nj + yy;
                acc = acc + xy;
            }
        }
    }
    __device__ __forceinline__ double key(double norm2) const {
#pragma clang fp contract(off)
        double k = acc;
        if (METRIC != 0) {
            const double den = sqrt(norm2) * sqrt(nj);
            k = -(acc / den);
        }
        return k == k ? k : (double)INFINITY;
    }
};
constexpr int VEC_MAX_D = 1024;   // own code in LDS: 8 KiB
// How the exact keys of knn_select's candidates read their codes: element by element, as whole vectors (above), or either.
enum KeyForm { KEYS_ELEMENTS, KEYS_VECTORS, KEYS_EITHER };
template <typename CT, int METRIC, int U>
__device__ __forceinline__ double exact_key_vec(const CT* cb, int vecs, const double* own, int j, double norm2) {
    constexpr int EPV = KeySum<CT, METRIC>::EPV;
    const vec4u* cj = reinterpret_cast<const vec4u*>(cb) + (int64_t)j * vecs;
    KeySum<CT, METRIC> sum;
    int c = 0;
    for (; c + U <= vecs; c += U) {
        vec4u v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = cj[c + u];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            sum.add(v[u], own + (c + u) * EPV);
            asm volatile("" : "+v"(sum.acc) : : "memory");   // the own code is read vector by vector, not all at once into registers
        }
    }
    if (c + 2 <= vecs) {
        const vec4u v0 = cj[c], v1 = cj[c + 1];
        sum.add(v0, own + c * EPV);
        sum.add(v1, own + (c + 1) * EPV);
        c += 2;
    }
    for (; c < vecs; ++c) sum.add(cj[c], own + c * EPV);
    return sum.key(norm2);
}
inline size_t own_code_bytes(int d, int vecs) { return vecs ? (size_t)d * sizeof(double) : 0; }
// The row's own code as doubles into LDS, by the whole workgroup (a barrier follows at the caller), and the sum of
// its squares in order.
template <typename CT>
__device__ __forceinline__ void own_code(const CT* row, int d, double* own, int tid, int threads) {
    for (int t = tid; t < d; t += threads) own[t] = (double)cb_f32<CT>(row, t);
}
__device__ __forceinline__ double own_norm2(const double* own, int d) {
#pragma clang fp contract(off)
    double n = 0.0;
    for (int t = 0; t < d; ++t) {
        const double xx = own[t] * own[t];
        n = n + xx;
    }
    return n;
}

// The approximate cosine keys are good to their error bound as long as a product of two coordinates that falls below
// the normal floats is nothing beside the codes' norms and no sum leaves the floats.  A code beyond
// COSINE_MIN .. COSINE_MAX (squared norm) leaves every row to the all-pairs pass, unless its exact keys do not
// depend on the norm: a code of zeros or with a coordinate that is no finite number has no similarity
// to any other.  n: the squared norm as computed in fp32.
constexpr float COSINE_MIN = 0x1p-100f, COSINE_MAX = 0x1p120f;
template <typename CT>
__device__ __forceinline__ bool cosine_in_doubt(const CT* code, int d, float n) {
    if (n >= COSINE_MIN && n <= COSINE_MAX) return false;
    bool nonzero = false;
    for (int t = 0; t < d; ++t) {
        const float x = cb_f32<CT>(code, t);
        if (!(fabsf(x) < INFINITY)) return false;
        nonzero |= x != 0.f;
    }
    return nonzero;
}

template <typename CT>
__global__ __launch_bounds__(NT) void knn_dist_direct(const CT* cb, int V, int d, int r0, int metric,
                                                      float* dist, int* doubt) {
    const int row = blockIdx.y;
    const int i = r0 + row;
    const int j = blockIdx.x * NT + threadIdx.x;
    if (j >= V) return;
    const CT* ci = cb + (int64_t)i * d;
    const CT* cj = cb + (int64_t)j * d;
    float key;
    if (metric == 0) {
        float acc = 0.f;
        for (int t = 0; t < d; ++t) {
            const float diff = cb_f32<CT>(ci, t) - cb_f32<CT>(cj, t);
            acc = fmaf(diff, diff, acc);
        }
        key = acc;
    } else {
        float ni = 0.f, nj = 0.f, dot = 0.f;
        for (int t = 0; t < d; ++t) {
            const float x = cb_f32<CT>(ci, t), y = cb_f32<CT>(cj, t);
            ni = fmaf(x, x, ni);
            nj = fmaf(y, y, nj);
            dot = fmaf(x, y, dot);
        }
        if (row == 0 && cosine_in_doubt(cj, d, nj)) *doubt = 1;   // every column of every row block
        key = -(dot / sqrtf(nj)) / sqrtf(ni);   // the product of the norms may leave the floats
    }
    dist[(int64_t)row * V + j] = key;
}


// ---- stage 1 (aligned shapes): approximate keys from a matrix-core contraction ----
// G = C C^T on MFMA 32x32 tiles with fp32 accumulation; squared l2 key
// n_i + n_j - 2 G_ij, cosine key -G_ij / sqrt(n_i n_j).  One wavefront owns a
// 64x64 block of the key matrix (2x2 MFMA tiles); a workgroup of 4 wavefronts
// owns 128x128.  Operand fragments are read straight from the codebook, which
// stays cache-resident (at most a few MB).
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// Sum of the squares of the coordinates held in 16 bytes of a row.
template <typename CT> __device__ __forceinline__ float sum_squares(const uint4& v, float n);
template <> __device__ __forceinline__ float sum_squares<float>(const uint4& v, float n) {
    const float x0 = __uint_as_float(v.x), x1 = __uint_as_float(v.y), x2 = __uint_as_float(v.z), x3 = __uint_as_float(v.w);
    return fmaf(x3, x3, fmaf(x2, x2, fmaf(x1, x1, fmaf(x0, x0, n))));
}
template <> __device__ __forceinline__ float sum_squares<uint16_t>(const uint4& v, float n) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float lo = __uint_as_float(w[q] << 16), hi = __uint_as_float(w[q] & 0xFFFF0000u);
        n = fmaf(hi, hi, fmaf(lo, lo, n));
    }
    return n;
}

// Whether fp32 values formed from a code are numbers whatever the other code: its squared norm n is moderate, and under
// the cosine key not zero.
__device__ __forceinline__ bool plain_code(float n, int metric) { return n < 0x1p120f && (metric == 0 || n > 0.f); }

// Squared norms of the rows (for the cosine key one over their roots: a product of two squared norms
// may leave the floats) and the largest squared norm, for rows that are whole 16-byte vectors at 16-byte
// aligned addresses.  *nmax is cleared beforehand; a norm is never below +0, so the bit patterns
// order like the values and an unsigned maximum collects it, asked for only by a workgroup that
// sees a smaller value there (a NaN norm is stored but left out of the maximum).  Rows of 256 bytes
// or more take a wavefront each, NORM_ROWS rows per workgroup with the loads of all of a
// wavefront's rows in flight together (index clamped, bits masked: no branch around a load);
// shorter rows take a thread each.
constexpr int NORM_ROWS = 32;
constexpr int NORM_WAVE_VECS = 16;
template <typename CT>
__global__ __launch_bounds__(NT) void knn_norms(const CT* cb, int V, int d, int metric, float* norms, float* nmax, int* doubt) {
    __shared__ float red[NW];
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x >> 6;
    const int vecs = d * (int)sizeof(CT) / 16;   // 16-byte vectors per row
    const uint4* cbv = reinterpret_cast<const uint4*>(cb);
    float m = 0.f;
    if (vecs >= NORM_WAVE_VECS) {
        constexpr int RPW = NORM_ROWS / NW;
        float n[RPW];
#pragma unroll
        for (int q = 0; q < RPW; ++q) n[q] = 0.f;
        for (int c0 = 0; c0 < vecs; c0 += WAVE) {
            const int c = c0 + lane;
            const uint32_t mask = c < vecs ? 0xFFFFFFFFu : 0u;
            const int cc = c < vecs ? c : vecs - 1;
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int i = blockIdx.x * NORM_ROWS + q * NW + w;
                uint4 v = cbv[(int64_t)(i < V ? i : V - 1) * vecs + cc];
                v.x &= mask; v.y &= mask; v.z &= mask; v.w &= mask;
                n[q] = sum_squares<CT>(v, n[q]);
            }
        }
        float t = 0.f;   // of the row that lane q finishes
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            const float sum = wave_sum(n[q]);
            if (lane == q) t = sum;
        }
        const int i = blockIdx.x * NORM_ROWS + lane * NW + w;
        if (lane < RPW && i < V) {
            norms[i] = metric == 0 ? t : rsqrtf(t);
            m = fmaxf(m, t);
            if (cosine_in_doubt(cb + (int64_t)i * d, d, t)) doubt[0] = 1;
            if (!plain_code(t, metric)) doubt[1] = 1;
        }
    } else {
        const int i = blockIdx.x * NT + threadIdx.x;
        if (i < V) {
            float n = 0.f;
            for (int c = 0; c < vecs; ++c) n = sum_squares<CT>(cbv[(int64_t)i * vecs + c], n);
            norms[i] = metric == 0 ? n : rsqrtf(n);
            if (cosine_in_doubt(cb + (int64_t)i * d, d, n)) doubt[0] = 1;
            if (!plain_code(n, metric)) doubt[1] = 1;
            m = fmaxf(m, n);
        }
    }
    m = fmaxf(wave_max(m), 0.f);
    if (lane == 0) red[w] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        float r = red[0];
        for (int v = 1; v < NW; ++v) r = fmaxf(r, red[v]);
        unsigned int* target = reinterpret_cast<unsigned int*>(nmax);
        const unsigned int bits = __float_as_uint(r);
        if (__hip_atomic_load(target, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < bits) atomicMax(target, bits);
    }
}

// Accumulator element r of lane l of a 32x32 MFMA tile is row 8*(r/4) + 4*(l/32) + r%4,
// column l%32 (rows come from the A operand, columns from the B operand).
// ni, nj: the two norms as knn_norms leaves them.
__device__ __forceinline__ float approx_key(float g, float ni, float nj, int metric) {
    return metric == 0 ? (ni + nj) - 2.f * g : -(g * nj) * ni;
}

// Columns are the VB tokens of the column operand (the codebook itself, or a sample of it) with
// norms nb; a row of dist holds VB keys.
__device__ __forceinline__ void store_tile(const f32x16& acc, int i0, int j0, int lane, int r0, int rows,
                                           int VB, int metric, const float* norms, const float* nb, float* dist) {
    const int j = j0 + (lane & 31);
    if (j >= VB) return;
    const float nj = nb[j];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int i = i0 + 8 * (r >> 2) + 4 * (lane >> 5) + (r & 3);
        if (i < r0 + rows) dist[(int64_t)(i - r0) * VB + j] = approx_key(acc[r], norms[i], nj, metric);
    }
}

// 64x64 block of G = A B^T for one wavefront: rows arow[0], arow[1] (32 each, one per lane & 31),
// columns brow[0], brow[1]; acc[a][b] is the 32x32 tile of row strip a and column strip b.
//
// bf16 codebook, d a multiple of 8: v_mfma_f32_32x32x16_bf16, 16 coordinates per step
// (lanes 0-31 carry coordinates k0..k0+7 of their row, lanes 32-63 k0+8..k0+15).
__device__ __forceinline__ void contract_block(const uint16_t* const (&arow)[2], const uint16_t* const (&brow)[2],
                                               int d, int lane, f32x16 (&acc)[2][2]) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    const int kh = 8 * (lane >> 5);
    for (int k0 = 0; k0 < d; k0 += 16) {
        const int kk = k0 + kh;
        uint4 fa[2], fb[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            if (kk < d) {
                fa[t] = *reinterpret_cast<const uint4*>(arow[t] + kk);
                fb[t] = *reinterpret_cast<const uint4*>(brow[t] + kk);
            } else {
                fa[t] = make_uint4(0, 0, 0, 0);
                fb[t] = fa[t];
            }
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8, fa[a]), __builtin_bit_cast(bf16x8, fb[b]), acc[a][b], 0, 0, 0);
    }
}

// fp32 codebook, d a multiple of 4: v_mfma_f32_32x32x2_f32, 2 coordinates per step
// (lanes 0-31 carry coordinate k, lanes 32-63 coordinate k+1); rows are read 8 floats at a time.
__device__ __forceinline__ void contract_block(const float* const (&arow)[2], const float* const (&brow)[2], int d,
                                               int lane, f32x16 (&acc)[2][2]) {
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    const bool hi = (lane >> 5) != 0;
    for (int k0 = 0; k0 < d; k0 += 8) {
        float4 fa[2][2], fb[2][2];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                if (k0 + 4 * h < d) {
                    fa[t][h] = *reinterpret_cast<const float4*>(arow[t] + k0 + 4 * h);
                    fb[t][h] = *reinterpret_cast<const float4*>(brow[t] + k0 + 4 * h);
                } else {
                    fa[t][h] = make_float4(0.f, 0.f, 0.f, 0.f);
                    fb[t][h] = fa[t][h];
                }
            }
#pragma unroll
        for (int s = 0; s < 4; ++s) {  // coordinates k0+2s, k0+2s+1
            float va[2], vb[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const float4 qa = fa[t][s >> 1], qb = fb[t][s >> 1];
                va[t] = (s & 1) ? (hi ? qa.w : qa.z) : (hi ? qa.y : qa.x);
                vb[t] = (s & 1) ? (hi ? qb.w : qb.z) : (hi ? qb.y : qb.x);
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x2f32(va[a], vb[b], acc[a][b], 0, 0, 0);
        }
    }
}

// The same block from packed operands (ap, bp: a lane's 16 bytes of step 0 of the two row strips and the
// two column strips).  acc holds what the products are added to.
template <typename CT>
__device__ __forceinline__ void mfma_step(const uint4& a, const uint4& b, f32x16& acc);
template <>
__device__ __forceinline__ void mfma_step<uint16_t>(const uint4& a, const uint4& b, f32x16& acc) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
template <>
__device__ __forceinline__ void mfma_step<float>(const uint4& a, const uint4& b, f32x16& acc) {
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.x), __uint_as_float(b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.y), __uint_as_float(b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.z), __uint_as_float(b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a.w), __uint_as_float(b.w), acc, 0, 0, 0);
}
template <typename CT>
__device__ __forceinline__ void contract_packed(const uint4* const (&ap)[2], const uint4* const (&bp)[2], int steps,
                                                f32x16 (&acc)[2][2]) {
    uint4 na[2] = {ap[0][0], ap[1][0]}, nb[2] = {bp[0][0], bp[1][0]};
    for (int s = 0; s < steps; ++s) {
        const uint4 fa[2] = {na[0], na[1]}, fb[2] = {nb[0], nb[1]};
        const int n = min(s + 1, steps - 1) * WAVE;   // the next step's operands are on their way meanwhile
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            na[t] = ap[t][n];
            nb[t] = bp[t][n];
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) mfma_step<CT>(fa[a], fb[b], acc[a][b]);
    }
}
__device__ __forceinline__ const uint4* packed_operand(const uint4* packed, int tile, int tiles, int steps, int lane) {
    return packed + ((int64_t)min(tile, tiles - 1) * steps * WAVE + lane);
}

// Keys of rows [r0, r0 + rows) to the S tokens of the sample, from packed operands; r0 is a multiple of
// 128.  blockIdx = (column tile, row tile).
template <typename CT>
__global__ __launch_bounds__(NT) void knn_sample_keys(const uint4* packed, const uint4* spacked, const float* norms,
                                                      const float* snorms, int V, int S, int steps, int r0, int rows,
                                                      int metric, float* skeys) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = threadIdx.x >> 6;
    const int i_base = r0 + blockIdx.y * 128 + (wave >> 1) * 64;
    const int j_base = blockIdx.x * 128 + (wave & 1) * 64;
    if (i_base >= r0 + rows || j_base >= S) return;
    const uint4* ap[2];
    const uint4* bp[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        ap[t] = packed_operand(packed, i_base / 32 + t, (int)packed_tiles(V), steps, lane);
        bp[t] = packed_operand(spacked, j_base / 32 + t, (int)packed_tiles(S), steps, lane);
    }
    f32x16 acc[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[a][b][r] = 0.f;
    contract_packed<CT>(ap, bp, steps, acc);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
            store_tile(acc[a][b], i_base + a * 32, j_base + b * 32, lane, r0, rows, S, metric, norms, snorms, skeys);
}

// All keys of rows [r0, r0 + rows) of the codebook cb (V tokens, norms `norms`) against the whole
// codebook into dist.  blockIdx = (column tile, row tile).
template <typename CT>
__global__ __launch_bounds__(NT) void knn_dist_mfma(const CT* cb, const float* norms, int V, int d, int r0, int rows,
                                                    int metric, float* dist) {
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = threadIdx.x >> 6;
    const int i_base = r0 + blockIdx.y * 128 + (wave >> 1) * 64;
    const int j_base = blockIdx.x * 128 + (wave & 1) * 64;
    if (i_base >= r0 + rows || j_base >= V) return;
    const CT* arow[2];
    const CT* brow[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        arow[t] = cb + (int64_t)min(i_base + t * 32 + (lane & 31), V - 1) * d;
        brow[t] = cb + (int64_t)min(j_base + t * 32 + (lane & 31), V - 1) * d;
    }
    f32x16 acc[2][2];
    contract_block(arow, brow, d, lane, acc);
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
            store_tile(acc[a][b], i_base + a * 32, j_base + b * 32, lane, r0, rows, V, metric, norms, norms, dist);
}

// Where the filtering contraction leaves a row block's candidates.
struct FilterOut {
    const float* thr;   // [rows] threshold of each row of the block, as a value (below)
    int* counts;        // [rows] keys at or below the threshold so far (may pass cap: the list is then cut)
    void* cand;         // [rows, cap] tokens or (order-preserving key, token), in no particular order
    int cap;
};
// The mask moved up by one, the freed bit set where the value lies below `least` (both numbers): a subtraction and
// its sign shifted in.  A compare would leave its result in scalar registers, which the next instruction may only
// read two cycles later.
__device__ __forceinline__ uint32_t shift_in_below(uint32_t mask, float value, float least) {
    return __builtin_amdgcn_alignbit(mask, __float_as_uint(value - least), 31);
}
// The same where a value or `least` may be no number, or both the same infinity: what does not compare is below.
__device__ __forceinline__ uint32_t shift_in_unless(uint32_t mask, float value, float least) {
    return (mask + mask) + (value >= least ? 0u : 1u);
}
// The filtering contraction takes the tokens as rows of its tiles and the query rows as columns: a
// lane then holds one query's values only, its threshold is one register, and a hit costs a compare.
// What is compared is not the key but its token-dependent part, larger for nearer tokens:
//   squared l2   v = G_ij - n_j / 2 (the matrix cores start from - n_j / 2),  key = n_i - 2 v
//   cosine       v = G_ij / sqrt(n_j),                                        key = - v / sqrt(n_i)
// fold[j]: - n_j / 2 or 1 / sqrt(n_j); NaN beyond the vocabulary, where v then passes no comparison.
// n in the functions: a norm as knn_norms leaves it (n_i, or 1 / sqrt(n_i)).
template <int METRIC>
__device__ __forceinline__ float fold_of(float n) { return METRIC == 0 ? -0.5f * n : n; }
template <int METRIC>
__device__ __forceinline__ float value_at(float key, float n) { return METRIC == 0 ? 0.5f * (n - key) : -key / n; }
template <int METRIC>
__device__ __forceinline__ float key_of_value(float v, float n) { return METRIC == 0 ? n - 2.f * v : -v * n; }
// Element r of a lane's column is token 8*(r/4) + 4*(lane/32) + r%4 of the tile: four loads of four.
__device__ __forceinline__ void load_fold(const float* fold, int tile, int lane, float (&o)[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float4 v = *reinterpret_cast<const float4*>(fold + tile * 32 + 8 * q + 4 * (lane >> 5));
        o[4 * q] = v.x; o[4 * q + 1] = v.y; o[4 * q + 2] = v.z; o[4 * q + 3] = v.w;
    }
}

// What the filtering contraction writes for a row.
enum ListForm {
    LIST_TOKENS,   // uint32 tokens
    LIST_PAIRS     // uint2 (order-preserving key, token)
};

// LDS of the filtering contraction.  A hit is staged as 512 * (row of the tile) + (token of the tile), the hits of a row
// next to each other, STAGE of them at a time.
template <int FORM>
struct FilterShared {
    static constexpr int STAGE = FORM == LIST_TOKENS ? FILTER_STAGE : 4096;
    int next[128];      // keys of the row kept; then the next free place among the tile's hits
    int start[128];     // first place of the row's hits
    int base[128];      // where they go in the row's list
    int total;
    uint16_t stage[STAGE];
    float value[FORM == LIST_PAIRS ? STAGE : 1];
    float norm[FORM == LIST_PAIRS ? 128 : 1];
};

// Filtering contraction: rows [r0, r0 + rows) against the whole codebook, keeping for every row
// only the tokens (and keys) at or below the row's threshold.  A workgroup owns a tile of 128
// rows by TT * 128 tokens.  It contracts, counts the kept keys per row in LDS, reserves each row's
// slots in its list with one atomic add per row, and stages the hits in LDS row by row, from where they are written
// out as runs (left to the lanes that found them, the writes were as many requests as hits, 26 million for
// V = 16384, k = 1000, and each hit cost a dozen instructions for its key and address).
// The reservation is on its way while the hits are staged (V = 40000, d = 64 bf16, k = 100: 1449 -> 1417 us the build).
// Grid: one-dimensional, 8 * ceil(row tiles / 8) * column tiles workgroups, dealt so that all
// column tiles of a row strip run on one XCD (workgroups go to the eight XCDs in turn) and a
// row's list and counter stay in that XCD's L2.
// A hit is a bit of a lane's mask: compare and shift in, two instructions a value.  Tokens alone are placed by walking
// the masks' bits, so several column tiles share one reservation; with keys, whose registers cannot be numbered at run
// time, by going over all 32 values, and the tile is one.
// V = 16384, d = 8 fp32, k = 1000: 193 us with hits written by the lanes that found them, 189 staged with their keys,
// 126 staged as tokens, 108 with 512 tokens to a tile and masks of shifted-in signs, 105 with the reservation on its way meanwhile.  V = 8192,
// d = 256 bf16, k = 100 (keys kept; bound by the operand loads): 78 -> 72.
typedef uint32_t tokens4 __attribute__((ext_vector_type(4), aligned(4)));
template <typename CT, int METRIC, int FORM, int TT>
__global__ __launch_bounds__(NT, 4) void knn_filter_list(const uint4* packed, const float* fold, const float* norms, int V,
                                                         int steps, int r0, int rows, const int* doubt, FilterOut f) {
    static_assert(TT == 1 || FORM == LIST_TOKENS, "keys stay in the accumulators until they are placed");
    static_assert(TT * 128 <= 512, "nine bits of a staged hit");
    constexpr int STAGE = FilterShared<FORM>::STAGE;
    __shared__ FilterShared<FORM> sh;
    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // its tiles' places in scalar registers: the cosine key spills otherwise
    const int nct = (V + 128 * TT - 1) / (128 * TT), nrt = (rows + 127) / 128;
    const int xcd = blockIdx.x & 7, q = blockIdx.x >> 3;
    const int ti = (q / nct) * 8 + xcd;
    const int tj = q % nct;
    if (ti >= nrt) return;   // the whole workgroup
    const int tiles = (int)packed_tiles(V);
    const int il_wg = ti * 128;        // first row of the workgroup within the block
    const int l_base = (wave >> 1) * 64;
    const bool plain = doubt[1] == 0;
    if (tid < 128) {
        sh.next[tid] = 0;
        if (FORM == LIST_PAIRS) sh.norm[tid] = norms[r0 + min(il_wg + tid, rows - 1)];
    }
    float least[2];                    // of the lane's two rows; beyond the block nothing is kept
    const uint4* bp[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int il = il_wg + l_base + b * 32 + (lane & 31);
        const float t = f.thr[min(il, rows - 1)];
        least[b] = il < rows ? t : plain ? INFINITY : NAN;
        bp[b] = packed_operand(packed, (r0 + il_wg + l_base) / 32 + b, tiles, steps, lane);
    }
    f32x16 acc[2][2];      // [token strip][query strip]
    uint32_t hits[TT][2];  // bit 31 - (16 a + r): element r of token strip a
#pragma unroll
    for (int c = 0; c < TT; ++c) {
        const int t_base = (tj * TT + c) * 4 + (wave & 1) * 2;   // first token tile
        hits[c][0] = hits[c][1] = 0u;
        if (t_base >= tiles) continue;                           // uniform
        const uint4* ap[2];
        float fd[2][16];
#pragma unroll
        for (int t = 0; t < 2; ++t) ap[t] = packed_operand(packed, t_base + t, tiles, steps, lane);
        if (METRIC == 0) {
#pragma unroll
            for (int a = 0; a < 2; ++a) load_fold(fold, min(t_base + a, tiles - 1), lane, fd[a]);
        }
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[a][b][r] = METRIC == 0 ? fd[a][r] : 0.f;
        contract_packed<CT>(ap, bp, steps, acc);
        if (METRIC != 0) {
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                load_fold(fold, min(t_base + a, tiles - 1), lane, fd[a]);
#pragma unroll
                for (int b = 0; b < 2; ++b)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[a][b][r] *= fd[a][r];
            }
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            uint32_t h = 0;
            if (plain) {
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int r = 0; r < 16; ++r) h = shift_in_below(h, acc[a][b][r], least[b]);
            } else {
#pragma unroll
                for (int a = 0; a < 2; ++a)
#pragma unroll
                    for (int r = 0; r < 16; ++r) h = shift_in_unless(h, acc[a][b][r], least[b]);
            }
            h = ~h;
            if ((t_base + 2) * 32 > V) {   // the last tiles: nothing beyond the vocabulary (nor strip 0 once more)
                const int left = V - t_base * 32 - 4 * (lane >> 5);
                for (int i = 0; i < 32; ++i)
                    if (i + (i & 28) >= left) h &= ~(0x80000000u >> i);
            }
            // the row itself is no candidate
            const int own = r0 + il_wg + l_base + b * 32 + (lane & 31) - t_base * 32;   // within the two strips?
            if ((unsigned)own < 64u && ((own >> 2) & 1) == (lane >> 5)) h &= ~(0x80000000u >> (4 * (own >> 3) + (own & 3)));
            hits[c][b] = h;
        }
    }
    __syncthreads();                   // the counters are cleared
    int mine[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        mine[b] = 0;
#pragma unroll
        for (int c = 0; c < TT; ++c) mine[b] += __popc(hits[c][b]);
        if (mine[b]) atomicAdd(&sh.next[l_base + b * 32 + (lane & 31)], mine[b]);
    }
    __syncthreads();
    int2 base = make_int2(0, 0);       // first wavefront: slots of two rows a lane, on their way while the hits are staged
    if (wave == 0) {                   // places of the rows' hits, and their slots in the lists; two rows a lane
        const int2 n = *reinterpret_cast<const int2*>(&sh.next[2 * lane]);   // above 0 only for rows of the block
        if (n.x > 0) base.x = atomicAdd(f.counts + il_wg + 2 * lane, n.x);
        if (n.y > 0) base.y = atomicAdd(f.counts + il_wg + 2 * lane + 1, n.y);
        const int incl = wave_scan_i<OpSum>(n.x + n.y, 0);
        const int2 at = make_int2(incl - n.x - n.y, incl - n.y);
        *reinterpret_cast<int2*>(&sh.start[2 * lane]) = at;
        *reinterpret_cast<int2*>(&sh.next[2 * lane]) = at;
        if (lane == WAVE - 1) sh.total = incl;
    }
    __syncthreads();
    const int total = sh.total;
    int place[2] = {0, 0};
#pragma unroll
    for (int b = 0; b < 2; ++b)
        if (mine[b]) place[b] = atomicAdd(&sh.next[l_base + b * 32 + (lane & 31)], mine[b]);
    if (FORM == LIST_TOKENS && total > STAGE) {
        // A dense tile (codes of one cluster next to each other in the codebook; uniform): every hit is placed by the lane
        // that holds it, four to a write.  Staged in rounds, such tiles are what the launch waits for: V = 8192, 512 codes
        // to a cluster, k = 100, 146 us against 30 (50 with a write for each hit), and 27 without clusters in order.
        if (wave == 0) *reinterpret_cast<int2*>(&sh.base[2 * lane]) = base;
        __syncthreads();
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int row = l_base + b * 32 + (lane & 31);
            int slot = sh.base[row] + place[b] - sh.start[row];
            uint32_t* lrow = static_cast<uint32_t*>(f.cand) + (int64_t)(il_wg + row) * f.cap;
#pragma unroll
            for (int c = 0; c < TT; ++c) {
                uint32_t h = hits[c][b];
                const uint32_t j0 = (uint32_t)(tj * (128 * TT) + c * 128 + (wave & 1) * 64 + 4 * (lane >> 5));
                auto next_token = [&]() -> uint32_t {
                    const int i = __clz((int)h);
                    h &= ~(0x80000000u >> i);
                    return j0 + i + (i & 28);
                };
                for (int n = __popc(h); n >= 4 && slot + 4 <= f.cap; n -= 4, slot += 4) {
                    const uint32_t t0 = next_token(), t1 = next_token(), t2 = next_token(), t3 = next_token();
                    *reinterpret_cast<tokens4*>(lrow + slot) = tokens4{t0, t1, t2, t3};
                }
                for (; h; ++slot) {
                    const uint32_t j = next_token();
                    if (slot < f.cap) lrow[slot] = j;
                }
            }
        }
        return;
    }
    for (int from = 0; from < total; from += STAGE) {   // once, unless more than STAGE pairs with keys are kept
        if (from) __syncthreads();
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            int at = place[b] - from;
#pragma unroll
            for (int c = 0; c < TT; ++c) {
                uint32_t h = hits[c][b];
                const int mark = (l_base + b * 32 + (lane & 31)) * 512 + c * 128 + (wave & 1) * 64 + 4 * (lane >> 5);
                const int n = __popc(h);
                if (at >= STAGE || at + n <= 0) {   // none of these in this round
                    at += n;
                    continue;
                }
                if (FORM == LIST_TOKENS) {
                    while (h) {
                        const int i = __clz((int)h);
                        h &= ~(0x80000000u >> i);
                        if ((unsigned)at < (unsigned)STAGE) sh.stage[at] = (uint16_t)(mark + i + (i & 28));
                        ++at;
                    }
                } else {
#pragma unroll
                    for (int a = 0; a < 2; ++a)
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if (h & (0x80000000u >> (16 * a + r))) {
                                if ((unsigned)at < (unsigned)STAGE) {
                                    sh.stage[at] = (uint16_t)(mark + 32 * a + 8 * (r >> 2) + (r & 3));
                                    sh.value[at] = acc[a][b][r];
                                }
                                ++at;
                            }
                }
            }
        }
        if (wave == 0 && from == 0) *reinterpret_cast<int2*>(&sh.base[2 * lane]) = base;
        __syncthreads();
        const int staged = min(total - from, STAGE);
        constexpr int BATCH = FORM == LIST_TOKENS ? 4 : 1;   // hits of a thread whose places are looked up together
        for (int e0 = tid; e0 < staged; e0 += BATCH * NT) {
            int hit[BATCH];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) hit[u] = sh.stage[min(e0 + u * NT, staged - 1)];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int e = e0 + u * NT, row = hit[u] >> 9;
                const int slot = sh.base[row] + (from + e - sh.start[row]);
                const uint32_t j = (uint32_t)(tj * (128 * TT) + (hit[u] & 511));
                if (e < staged && slot < f.cap) {
                    const int64_t at = (int64_t)(il_wg + row) * f.cap + slot;
                    if (FORM == LIST_TOKENS) {
                        static_cast<uint32_t*>(f.cand)[at] = j;
                    } else {
                        const float key = key_of_value<METRIC>(sh.value[e], sh.norm[row]);
                        static_cast<uint2*>(f.cand)[at] = make_uint2(min(ord_key(key), 0xFFFFFFFEu), j);
                    }
                }
            }
        }
    }
}

// ---- sampled thresholds ----
// Token of sample slot s: one token out of each of S equal strata of the vocabulary, at a hashed
// place inside the stratum.
__host__ __device__ inline int sample_token(int s, int S, int V) {
    const uint32_t h = ((uint32_t)s * 2654435761u) >> 16;   // 16 hashed bits
    const int64_t j = ((int64_t)s * V + (((int64_t)h * V) >> 16)) / S;
    return j < V ? (int)j : V - 1;
}

// The packed operands of the codebook (its `tiles` tiles) and, after them, of the sample; one thread per
// lane of a step.  Also fold[] for every token of those tiles, and the sample's fold and norms.
template <typename CT, int METRIC>
__global__ __launch_bounds__(NT) void knn_pack(const CT* cb, const float* norms, int V, int d, int S, int steps,
                                               uint4* packed, uint4* spacked, float* fold, float* sfold, float* snorms) {
    const int tiles = (int)packed_tiles(V), stiles = (int)packed_tiles(S);
    const int64_t t = (int64_t)blockIdx.x * NT + threadIdx.x;
    const int lane = (int)(t & (WAVE - 1));
    const int64_t unit = t >> 6;
    const int step = (int)(unit % steps);
    const int64_t tile = unit / steps;
    if (tile >= tiles + stiles) return;
    const bool of_sample = tile >= tiles;
    const int slot = (int)(of_sample ? tile - tiles : tile) * 32 + (lane & 31);
    const bool there = slot < (of_sample ? S : V);
    const int j = !there ? 0 : of_sample ? sample_token(slot, S, V) : slot;
    const CT* row = cb + (int64_t)j * d;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (there) {
        if constexpr (sizeof(CT) == 2) {
            const int c = step * 16 + 8 * (lane >> 5);
            if (c < d) v = *reinterpret_cast<const uint4*>(row + c);   // d is a multiple of 8
        } else {
            const uint32_t* w = reinterpret_cast<const uint32_t*>(row) + step * 8 + (lane >> 5);
            const int left = d - step * 8;   // 4 or at least 8
            v.x = w[0];
            v.y = w[2];
            if (left > 4) { v.z = w[4]; v.w = w[6]; }
        }
    }
    (of_sample ? spacked + (unit - (int64_t)tiles * steps) * WAVE : packed + unit * WAVE)[lane] = v;
    if (step == 0 && lane < 32) {
        if (!of_sample) fold[slot] = there ? fold_of<METRIC>(norms[slot]) : NAN;
        else if (there) {
            snorms[slot] = norms[j];
            sfold[slot] = fold_of<METRIC>(norms[j]);
        }
    }
}

// One wavefront per row: a value with between rank and rank + slack of the row's S <= 64 * NS = 4096 keys
// to the sample at or below it (bisection over the integer range of the keys, each step one
// count) becomes the row's threshold (as the value that the filtering contraction compares); the row's list length is
// cleared.  For samples beyond what knn_thresholds holds.
// (At most four wavefronts per SIMD are aimed at: with more as its goal the compiler's scheduler
// keeps the register count down by waiting for each of the 64 loads in turn.)
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(1, 4))) void knn_sample_rank(const float* skeys, int S, int rows, int rank, int slack,
                                                      const float* norms, int r0, int metric, float* thr, int* counts) {
    constexpr int NS = 64;
    const int lane = threadIdx.x & (WAVE - 1);
    const int row = blockIdx.x * NW + (threadIdx.x >> 6);
    if (row >= rows) return;   // whole wavefronts leave; no workgroup barrier below
    const float* krow = skeys + (int64_t)row * S;
    uint32_t keys[NS];
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
#pragma unroll
    for (int e = 0; e < NS; ++e) {
        const int sidx = e * WAVE + lane;
        // no branch and no select on the loaded value, so that all loads are in flight together:
        // beyond the sample the index is clamped and the key forced to all ones by a mask
        const uint32_t beyond = (uint32_t)((S - 1 - sidx) >> 31);
        const float v = krow[min(sidx, S - 1)];
        keys[e] = min(ord_key(v), 0xFFFFFFFEu) | beyond;
        kmin = min(kmin, keys[e]);
        kmax = max(kmax, keys[e] & ~beyond);
    }
    kmin = (uint32_t)__builtin_amdgcn_readlane(wave_scan_i<OpMin>((int)(kmin ^ 0x80000000u), INT_MAX), 63) ^ 0x80000000u;
    kmax = (uint32_t)__builtin_amdgcn_readlane(wave_scan_i<OpMax>((int)(kmax ^ 0x80000000u), INT_MIN), 63) ^ 0x80000000u;
    // count(lo) < rank <= count(hi)
    int64_t lo = (int64_t)kmin - 1, hi = (int64_t)kmax;
    while (hi - lo > 1) {
        const int64_t mid64 = lo + ((hi - lo) >> 1);
        const uint32_t mid = (uint32_t)mid64;
        int c = 0;
#pragma unroll
        for (int e = 0; e < NS; ++e) c += keys[e] <= mid ? 1 : 0;
        c = __builtin_amdgcn_readlane(wave_scan_i<OpSum>(c, 0), 63);
        if (c < rank) {
            lo = mid64;
        } else {
            hi = mid64;
            if (c <= rank + slack) break;
        }
    }
    if (lane == 0) {
        const float key = ord_inv((uint32_t)hi), n = norms[r0 + row];
        thr[row] = metric == 0 ? value_at<0>(key, n) : value_at<1>(key, n);
        counts[row] = 0;
    }
}

// Thresholds of 32 rows per workgroup of sixteen wavefronts, from the rows' values to the sample (what the filtering
// contraction compares: larger for nearer tokens).  A wavefront holds the values to its part of the S <= 512 TPW
// sampled tokens in the accumulators, a lane those of one row (and another lane the other half): the sample's keys
// never leave the registers.  Searched is a value with between rank and rank + slack of a row's sample values at or
// above it; every step counts (two instructions a value, a subtraction and its sign shifted into a mask: a compare and an addition
// of its bit would have to wait for each other through the scalar registers) and adds up over the wavefronts through LDS.  The first
// guesses are those of a normal distribution with the values' mean and variance (z, per_count: its quantile for the
// wanted count and the step per count there, in standard deviations), as long as they fall between what is known;
// after three of them, or when they do not, the interval's integer image is halved, which always ends.
// Bound by the counts' issue and the operands; V = 16384, d = 8 fp32, S = 2048: 34 us against 82 for a
// contraction that wrote the keys (47) and a kernel that ranked them by halving alone (35).
constexpr int THR_THREADS = 1024;
constexpr int THR_WAVES = THR_THREADS / WAVE;
template <typename CT, int METRIC, int TPW>
__global__ __launch_bounds__(THR_THREADS, 4) void knn_thresholds(const uint4* packed, const uint4* spacked, const float* sfold,
                                                                 int V, int S, int steps, int r0, int rows, int rank,
                                                                 int slack, float z, float per_count, const int* doubt,
                                                                 float* least, int* counts) {
    __shared__ float4 stat[THR_WAVES][32];      // per wavefront and row: sum, sum of squares, least, greatest
    __shared__ int found[2][THR_WAVES][32];
    const int lane = threadIdx.x & (WAVE - 1);
    const int wave = threadIdx.x >> 6;
    const int q = lane & 31;                    // row of the strip
    const int i0 = r0 + blockIdx.x * 32;
    const int tiles = S / 32;                   // S is a multiple of 64
    const int t0 = wave * TPW;
    const int mine = min(max(tiles - t0, 0), TPW);   // tiles of this wavefront
    const bool plain = doubt[1] == 0;
    f32x16 acc[TPW];
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
        float fd[16];
        load_fold(sfold, min(t0 + u, tiles - 1), lane, fd);
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[u][r] = METRIC == 0 ? fd[r] : 0.f;
    }
    {
        const uint4* bp = packed_operand(packed, i0 / 32, (int)packed_tiles(V), steps, lane);
        const uint4* ap[TPW];
#pragma unroll
        for (int u = 0; u < TPW; ++u) ap[u] = packed_operand(spacked, t0 + u, tiles, steps, lane);
        uint4 nb = bp[0], na[TPW];
#pragma unroll
        for (int u = 0; u < TPW; ++u) na[u] = ap[u][0];
        for (int st = 0; st < steps; ++st) {
            const uint4 b = nb;
            uint4 a[TPW];
            const int n = min(st + 1, steps - 1) * WAVE;   // the next step's operands are on their way meanwhile
            nb = bp[n];
#pragma unroll
            for (int u = 0; u < TPW; ++u) {
                a[u] = na[u];
                na[u] = ap[u][n];
            }
#pragma unroll
            for (int u = 0; u < TPW; ++u) mfma_step<CT>(a[u], b, acc[u]);
        }
    }
    float sum = 0.f, squares = 0.f, low = INFINITY, high = neg_inf_f();
#pragma unroll
    for (int u = 0; u < TPW; ++u) {
        if (u < mine) {                         // uniform
            if (METRIC != 0) {
                float fd[16];
                load_fold(sfold, t0 + u, lane, fd);
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[u][r] *= fd[r];
            }
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float v = acc[u][r];
                sum += v;
                squares = fmaf(v, v, squares);
                low = fminf(low, v);
                high = fmaxf(high, v);
            }
        }
    }
    sum += __shfl_xor(sum, 32, WAVE);
    squares += __shfl_xor(squares, 32, WAVE);
    low = fminf(low, __shfl_xor(low, 32, WAVE));
    high = fmaxf(high, __shfl_xor(high, 32, WAVE));
    if (lane < 32) stat[wave][q] = make_float4(sum, squares, low, high);
    __syncthreads();
    sum = squares = 0.f;
    low = INFINITY;
    high = neg_inf_f();
#pragma unroll
    for (int w = 0; w < THR_WAVES; ++w) {
        const float4 x = stat[w][q];
        sum += x.x;
        squares += x.y;
        low = fminf(low, x.z);
        high = fmaxf(high, x.w);
    }
    const float mean = sum / (float)S;
    const float sd = sqrtf(fmaxf(squares / (float)S - mean * mean, 0.f));
    // values as ordered integers: count(lo) >= rank (as far as is known), count(hi) < rank.  No number among a row's
    // values: an empty interval, and a threshold that leaves the list empty; the row is then flagged.
    int64_t lo = (int64_t)ord_key(low), hi = (int64_t)ord_key(high) + 1;
    float guess = mean + z * sd;
    bool done = hi - lo <= 1;
    for (int pass = 0; __any(!done); ++pass) {  // the same in every wavefront: all hold the same rows' state
        int64_t at = (int64_t)ord_key(guess);
        if (pass >= 4 || !(at > lo && at < hi)) at = lo + ((hi - lo) >> 1);
        const float t = ord_inv((uint32_t)at);
        int c = 16 * mine;
#pragma unroll
        for (int u = 0; u < TPW; ++u)
            if (u < mine) {
                uint32_t below = 0;
                if (plain) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) below = shift_in_below(below, acc[u][r], t);
                } else {
#pragma unroll
                    for (int r = 0; r < 16; ++r) below = shift_in_unless(below, acc[u][r], t);
                }
                c -= __popc(below);
            }
        c += __shfl_xor(c, 32, WAVE);
        if (lane < 32) found[pass & 1][wave][q] = c;
        __syncthreads();                        // one barrier a pass: the buffers alternate
        c = 0;
#pragma unroll
        for (int w = 0; w < THR_WAVES; ++w) c += found[pass & 1][w][q];
        if (!done) {
            if (c >= rank) {
                lo = at;
                done = c <= rank + slack;
            } else {
                hi = at;
            }
            done |= hi - lo <= 1;
            guess = t + ((float)(c - rank) - 0.5f * (float)slack) * per_count * sd;
        }
    }
    const int row = blockIdx.x * 32 + q;
    if (wave == 0 && lane < 32 && row < rows) {
        least[row] = ord_inv((uint32_t)lo);
        counts[row] = 0;
    }
}

// ---- stage 2: select, re-rank exactly, emit ----
constexpr int CROWDED = 64;   // candidates in one bucket above which a row takes the sorting network
constexpr int NARROW_THREADS = 128;   // threads per row where at most 256 candidates are wanted of a list
constexpr int SEL_MAXW = 8;   // wavefronts of the largest selection workgroup (512 threads)
template <int CAP, int TNT>
struct SelectShared {
    static_assert(CAP % 128 == 0, "lds_slot permutes blocks of 128 slots");
    // Buckets of the two histograms, 16-bit counters (then starts) two to a word.
    static constexpr int BUCKETS = CAP >= 1024 ? 2048 : (2 * TNT > 512 ? 2 * TNT : 512);
    double key[CAP];   // both indexed by lds_slot in the sorting network, plainly by the buckets
    int idx[CAP];
    uint32_t hist[BUCKETS / 2];
    unsigned red_u[2 * SEL_MAXW];
    int red_c[2][SEL_MAXW];   // per-wavefront counts of a counting pass, double-buffered
    int cut[3];               // boundary bucket, keys up to and including it; crowded buckets seen
    int taken;                // candidates so far
    unsigned thr_max;         // the largest approximate key among them
    double last;              // exact key of the last token emitted
};

// Exclusive starts from the counts in h (BUCKETS 16-bit counters, two to a word), in place, by the
// whole workgroup; every thread holds BUCKETS / TNT consecutive buckets in registers meanwhile.
// red: one word per wavefront.  each(bucket, start, count) is run for every bucket of the thread.  The caller's barriers
// stand before (counts complete) and after (starts visible).
template <int BUCKETS, int TNT, typename F>
__device__ __forceinline__ void bucket_starts(uint32_t* h, int* red, int tid, F each) {
    constexpr int W = BUCKETS / 2 / TNT;
    static_assert(W >= 1, "a thread owns whole words");
    uint32_t w[W];
    int sum = 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        w[q] = h[tid * W + q];
        sum += (int)(w[q] & 0xFFFFu) + (int)(w[q] >> 16);
    }
    const int incl = wave_scan_i<OpSum>(sum, 0);
    if ((tid & (WAVE - 1)) == WAVE - 1) red[tid >> 6] = incl;
    __syncthreads();
    int at = incl - sum;
#pragma unroll
    for (int v = 0; v < TNT / WAVE; ++v) at += v < (tid >> 6) ? red[v] : 0;
#pragma unroll
    for (int q = 0; q < W; ++q) {
        const int c0 = (int)(w[q] & 0xFFFFu), c1 = (int)(w[q] >> 16);
        each(2 * (tid * W + q), at, c0);
        each(2 * (tid * W + q) + 1, at + c0, c1);
        h[tid * W + q] = (uint32_t)at | ((uint32_t)(at + c0) << 16);
        at += c0 + c1;
    }
}
__device__ __forceinline__ int bucket_start(const uint32_t* h, int b) { return (int)((h[b >> 1] >> (16 * (b & 1))) & 0xFFFFu); }
__device__ __forceinline__ int bucket_add(uint32_t* h, int b) {   // what the counter held before
    return (int)((atomicAdd(&h[b >> 1], 1u << (16 * (b & 1))) >> (16 * (b & 1))) & 0xFFFFu);
}

// The candidates of the buckets, ranked: `count` of them in sh.key, sh.idx, those of a bucket next to each other.  A
// candidate's rank is its bucket's start plus the smaller ones in the bucket.  The first `need` are written.
template <int BUCKETS, int TNT, int CAP, typename SH, typename F>
__device__ __forceinline__ void rank_in_buckets(SH& sh, int count, int need, int tid, F bucket_of, int32_t* orow) {
    constexpr int PT = CAP > TNT ? CAP / TNT : 1;
    double key[PT];
    int from[PT], to[PT];
#pragma unroll
    for (int e = 0; e < PT; ++e) key[e] = sh.key[min(e * TNT + tid, count - 1)];   // in flight together
#pragma unroll
    for (int e = 0; e < PT; ++e) {
        const int b = bucket_of(key[e]);
        from[e] = bucket_start(sh.hist, b);
        to[e] = min(b + 1 < BUCKETS ? bucket_start(sh.hist, b + 1) : count, count);
    }
#pragma unroll
    for (int e = 0; e < PT; ++e) {
        const int p = e * TNT + tid;
        if (p < count) {
            const int tok = sh.idx[p];
            int rank = from[e], equal = 0;
            for (int q = from[e]; q < to[e]; ++q) {
                const double kq = sh.key[q];
                rank += kq < key[e] ? 1 : 0;
                equal += kq == key[e] ? 1 : 0;
            }
            if (equal > 1)   // in the order of their tokens
                for (int q = from[e]; q < to[e]; ++q) rank += (int)((sh.key[q] == key[e]) & (sh.idx[q] < tok));
            // a row that fails the proof is written again by the all-pairs pass
            if (rank < need) orow[1 + rank] = tok;
            if (rank == need - 1) sh.last = key[e];
        }
    }
}
// The candidates in sh.key, sh.idx (in any order) sorted by (key, token); the first `need` are written.
template <int TNT, typename SH>
__device__ __forceinline__ void sort_candidates(SH& sh, int count, int need, int tid, int32_t* orow) {
    int P = 4;   // the sort takes four elements per thread
    while (P < count) P <<= 1;
    for (int c = count + tid; c < P; c += TNT) {
        sh.key[c] = INFINITY;
        sh.idx[c] = INT_MAX;
    }
    // the slots' first contents may be in any order
    struct Cand {
        double key;
        int idx;
    };
    bitonic_sort_lds<TNT, Cand>(
        P, tid, [&](int p) { return Cand{sh.key[p], sh.idx[p]}; },
        [&](int p, const Cand& c) { sh.key[p] = c.key; sh.idx[p] = c.idx; },
        [](const Cand& a, const Cand& b) { return (a.key > b.key) | ((a.key == b.key) & (a.idx > b.idx)); },
        [](bool sw, const Cand& a, const Cand& b) { return Cand{sw ? b.key : a.key, sw ? b.idx : a.idx}; });
    for (int s = tid; s < need; s += TNT) orow[1 + s] = sh.idx[lds_slot(s)];
    if (tid == 0) sh.last = sh.key[lds_slot(need - 1)];
}

// Whether no discarded token can belong to the row: each has an approximate key of at least thr, hence an exact key
// of at least thr less the approximation's error; the last token taken (exact key `last`) must lie at or below that.
__device__ __forceinline__ bool proven(double last, float thr, int d, int metric, float err_rel, float err_abs, float err_norm,
                                       float norm, float nmax, bool by_norms) {
    bool ok = true;
    // products and sums below the normal floats may lose up to the smallest of those each
    double eabs = (double)err_abs + (metric == 0 ? (d + 8) * 0x1p-124 : 0.0);
    if (by_norms) {
        // Squared l2: the error of a key grows with the norms of its two codes, and the bound needs the
        // largest norm a discarded token can have.  A token with norm n_j > 4 (n_i + last) is further
        // away than the last one taken whatever its approximate key says, since |c_i - c_j|^2 >=
        // (sqrt n_j - sqrt n_i)^2 > (2 sqrt(n_i + last) - sqrt n_i)^2 >= last; so only norms up to that
        // (taken a thousandth larger, for the rounding of the fp32 norms) have to be covered.  A few
        // codes of very large norm then no longer send every row to the all-pairs pass.
        const double ni = (double)norm;
        const double far = 4.004 * (ni + last);
        const double nbound = far < (double)nmax ? far : (double)nmax;   // far may be inf or NaN: then the maximum
        eabs += (double)err_norm * (ni + nbound);
        if (!(ni < 0x1p120)) ok = false;
    }
    const double num = (double)thr - eabs;
    const double floor_discarded = num - 1.01 * (double)err_rel * fabs(num);
    // Squared l2 beyond the floats: a discarded token may have an approximate key that is infinite or no number.
    // Its code or the difference then has a square of about 2^127 or more, or a coordinate that is no
    // finite number, and with the row's own norm below 2^120 its exact key lies above 2^126.
    return ok && last <= floor_discarded && (metric != 0 || thr < 0x1p124f);
}

// Error model of the approximate keys:
//   |approximate - exact| <= err_rel * |exact| + err_abs + err_norm * (norm_i + max norm)
// (the last term applies when norms is not null: keys formed as n_i + n_j - 2 G_ij).
//
// NK > 0: the row's V <= NK * TNT approximate keys (TNT threads per row) are held in registers as order-preserving
// unsigned integers; NK == 0: they are re-read from the workspace in every pass.
// A threshold with between k-1+pad and `fit` keys at or below it is found by bisection over the
// keys' integer range, every step one counting pass over the registers (compare, add, one
// reduction); a list first narrows that range to one bucket of a histogram of its keys.
// Runs body(e) for every key slot of a thread: fully unrolled when the keys sit in registers.
template <int NK, typename F>
__device__ __forceinline__ void for_keys(int npt, F body) {
    if (NK > 0) {
#pragma unroll
        for (int e = 0; e < NK; ++e) body(e);
    } else {
        for (int e = 0; e < npt; ++e) body(e);
    }
}

//
// LIST: the row's keys are not a row of the key block but its candidate list of the filtering
// contraction, list.counts[row] pairs (key, token) with NK * TNT >= list.cap; every token not on
// the list has an approximate key above every key on it, so the proof below reads the same.  A
// list that was cut at its capacity, is longer than the registers hold (the proof takes every listed
// token for seen), or is shorter than the selection wants, flags the row.
//
// KEYS: how the candidates' exact keys read their codes.  Both forms in one kernel cost registers, and short codes gain nothing by vectors: so
// selections from whole rows are kernels of one form each (which one: row_vecs at the launch).  Builds before exact keys by vectors /
// with both forms in every kernel / now: V = 8192, d = 8 fp32, k = 30, cosine 201.5 / 204.7 / 201.5 us; V = 4000, d = 8 bf16, k = 300
// 77.7 / 80.0 / 78.1; V = 1024, d = 9, k = 700 34.9 / 36.6 / 34.7.
template <typename CT, int NK, int CAP, int TNT, bool LIST, int KEYS>
__global__ __launch_bounds__(TNT, NK >= 64 ? 4 : !LIST ? 8 : NK == 32 ? 5 : (CAP > 256 || NK == 24) ? 6 : 8) void knn_select(const CT* cb, int V, int d, int k, int metric, int r0,
                                                 const float* dist, FilterOut list, float err_rel, float err_abs,
                                                 float err_norm, const float* norms, const float* nmax,
                                                 const int* doubt, int32_t* out, int* flags, int vecs_or_0) {
    static_assert(!LIST || NK > 0, "a candidate list is held in registers");
    constexpr int TNW = TNT / WAVE;
    using Shared = SelectShared<CAP, TNT>;
    __shared__ Shared sh;
    extern __shared__ __align__(16) double own[];   // vecs > 0: the row's own code
    const int vecs = KEYS == KEYS_ELEMENTS ? 0 : vecs_or_0;
    const int row = blockIdx.x;
    const int i = r0 + row;
    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1);
    const int wave = tid >> 6;
    const float* drow = LIST ? nullptr : dist + (int64_t)row * V;
    int32_t* orow = out + (int64_t)i * k;
    const int need = k - 1;
    // rows of four-coordinate groups, each group one aligned load (16 bytes fp32, 8 bytes bf16)
    const bool vec4 = (d % 4 == 0) && ((reinterpret_cast<uintptr_t>(cb) & 15) == 0);
    if (tid == 0) {
        orow[0] = i;
        flags[row] = 0;
        sh.cut[2] = 0;
        sh.taken = 0;
        sh.thr_max = 0u;
        sh.last = INFINITY;
    }
    if (need == 0) return;
    const int pad = 8 + need / 128;
    const int want = min(V - 1, need + pad);
    if (want > CAP || (metric != 0 && *doubt)) {
        if (tid == 0) flags[row] = 1;
        return;
    }

    constexpr int NKR = NK > 0 ? NK : 1;
    uint32_t keys[NKR];
    uint32_t toks[LIST ? NKR : 1];
    const int npt = NK > 0 ? NK : (V + TNT - 1) / TNT;   // keys per thread
    const int listed = LIST ? list.counts[row] : 0;
    if (LIST && (listed > min(list.cap, NK * TNT) || listed < want)) {
        if (tid == 0) flags[row] = 1;
        return;
    }
    // Token of element e of this thread.  Keys in registers: groups of four consecutive tokens per
    // thread, (e / 4) * TNT + tid being the group, so that a group is one 16-byte load; else e * TNT + tid.
    auto token_of = [&](int e) -> int {
        if (LIST) return (int)toks[e];
        return NK > 0 ? (((e >> 2) * TNT + tid) << 2) + (e & 3) : e * TNT + tid;
    };
    // key of element e; 0xFFFFFFFF for the row's own token and padding
    auto key_at = [&](int e) -> uint32_t {
        if (NK > 0) return keys[e];
        const int j = e * TNT + tid;
        return (j < V && j != i) ? min(ord_key(drow[j]), 0xFFFFFFFEu) : 0xFFFFFFFFu;
    };
    if (LIST) {
        const uint2* lrow = static_cast<const uint2*>(list.cand) + (int64_t)row * list.cap;
#pragma unroll
        for (int e = 0; e < NKR; ++e) {
            const int slot = e * TNT + tid;
            const uint2 q = lrow[slot < listed ? slot : listed - 1];   // no branch: all loads in flight together (listed >= 1)
            keys[e] = slot < listed ? q.x : 0xFFFFFFFFu;
            toks[e] = q.y;
        }
    } else if (NK > 0) {
        if ((V & 3) == 0) {   // every row of the key block starts 16-byte aligned and ends with a whole group
            // No branch and no select on a loaded value, so that all the row's loads are in flight
            // together: a group beyond the row re-reads the last one, and its keys, like the row's own
            // token's, are forced to all ones by a mask.
            float4 q[NKR / 4 > 0 ? NKR / 4 : 1];
#pragma unroll
            for (int g = 0; g < NKR / 4; ++g)
                q[g] = *reinterpret_cast<const float4*>(drow + min((g * TNT + tid) << 2, V - 4));
#pragma unroll
            for (int g = 0; g < NKR / 4; ++g) {
                const int j0 = (g * TNT + tid) << 2;
                const float f[4] = {q[g].x, q[g].y, q[g].z, q[g].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int j = j0 + e;
                    const uint32_t out = (uint32_t)((V - 1 - j) >> 31) | (uint32_t)(-(int)(j == i));
                    keys[4 * g + e] = min(ord_key(f[e]), 0xFFFFFFFEu) | out;
                }
            }
        } else {
#pragma unroll
            for (int g = 0; g < NKR / 4; ++g) {
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int j = ((g * TNT + tid) << 2) + e;
                    const float f = j < V ? drow[j] : 0.f;
                    keys[4 * g + e] = (j < V && j != i) ? min(ord_key(f), 0xFFFFFFFEu) : 0xFFFFFFFFu;
                }
            }
        }
    }

    if (CAP <= 1024 && (KEYS == KEYS_VECTORS || vecs)) own_code<CT>(cb + (int64_t)i * d, d, own, tid, TNT);
    // range of the keys
    for (int w = tid; w < Shared::BUCKETS / 2; w += TNT) sh.hist[w] = 0u;
    uint32_t kmin = 0xFFFFFFFFu, kmax = 0u;
    for_keys<NK>(npt, [&](int e) {
        const uint32_t key = key_at(e);
        if (key != 0xFFFFFFFFu) { kmin = min(kmin, key); kmax = max(kmax, key); }
    });
    // unsigned order through signed scans: flip the top bit
    kmin = (uint32_t)__builtin_amdgcn_readlane(wave_scan_i<OpMin>((int)(kmin ^ 0x80000000u), INT_MAX), 63) ^ 0x80000000u;
    kmax = (uint32_t)__builtin_amdgcn_readlane(wave_scan_i<OpMax>((int)(kmax ^ 0x80000000u), INT_MIN), 63) ^ 0x80000000u;
    if (lane == 0) { sh.red_u[wave] = kmin; sh.red_u[TNW + wave] = kmax; }
    __syncthreads();
    kmin = sh.red_u[0]; kmax = sh.red_u[TNW];
#pragma unroll
    for (int w = 1; w < TNW; ++w) { kmin = min(kmin, sh.red_u[w]); kmax = max(kmax, sh.red_u[TNW + w]); }

    // Whole rows: aim at a count of at most the power of two that holds `want`.  Lists, whose
    // histogram below leaves few keys beyond `want`: at what the LDS holds.
    int fit = 1;
    while (fit < want) fit <<= 1;
    if (LIST || fit > CAP) fit = CAP;
    // Bisection over [kmin - 1, kmax] (as 64-bit integers): count(lo) < want <= count(hi).  The best
    // threshold seen is kept: the one with the fewest keys at or below it that still has `want` and
    // fits the LDS; the search stops as soon as that number is at most `fit`.
    int64_t lo = (int64_t)kmin - 1, hi = (int64_t)kmax;
    uint32_t thr_key = kmax;
    int best = LIST ? listed : V - 1;   // count(kmax): every listed token, every other token
    if (LIST) {
        // One histogram over the keys' range narrows the search to the bucket in which the count passes
        // `want`: a dozen counting passes, each a reduction and a barrier, become one.
        const int span_bits = 32 - __clz((int)(kmax - kmin));
        constexpr int LOG_BUCKETS = 31 - __builtin_clz(Shared::BUCKETS);
        const int shift = span_bits > LOG_BUCKETS ? span_bits - LOG_BUCKETS : 0;
#pragma unroll
        for (int e = 0; e < NKR; ++e)
            if (keys[e] != 0xFFFFFFFFu) bucket_add(sh.hist, (int)((keys[e] - kmin) >> shift));
        __syncthreads();
        bucket_starts<Shared::BUCKETS, TNT>(sh.hist, sh.red_c[0], tid, [&](int bucket, int start, int n) {
            if (start < want && start + n >= want) {
                sh.cut[0] = bucket;
                sh.cut[1] = start + n;
            }
        });
        __syncthreads();
        lo = (int64_t)kmin + ((int64_t)sh.cut[0] << shift) - 1;   // below the bucket: fewer than `want`
        const int64_t top = (int64_t)kmin + ((int64_t)(sh.cut[0] + 1) << shift) - 1;
        hi = top < hi ? top : hi;
        best = sh.cut[1];
        thr_key = (uint32_t)hi;
        for (int w = tid; w < Shared::BUCKETS / 2; w += TNT) sh.hist[w] = 0u;   // every count has been read before the barrier above; used again after two more
    }
    for (int pass = 0; pass < 40 && best > fit && hi - lo > 1; ++pass) {
        const int64_t mid64 = lo + ((hi - lo) >> 1);
        const uint32_t mid = (uint32_t)mid64;
        int c = 0;
        for_keys<NK>(npt, [&](int e) { c += key_at(e) <= mid ? 1 : 0; });   // own token and padding: 0xFFFFFFFF > mid
        c = __builtin_amdgcn_readlane(wave_scan_i<OpSum>(c, 0), 63);
        if (lane == 0) sh.red_c[pass & 1][wave] = c;
        __syncthreads();         // one barrier per pass: the buffers alternate
        c = 0;
#pragma unroll
        for (int w = 0; w < TNW; ++w) c += sh.red_c[pass & 1][w];
        if (c < want) {
            lo = mid64;
        } else {   // counts grow with the threshold: c <= best = count(hi)
            hi = mid64;
            best = c;
            thr_key = mid;
        }
    }
    if (best > CAP) {            // more (nearly) equal keys around the threshold than the LDS holds
        if (tid == 0) flags[row] = 1;
        return;
    }

    // compaction of every j != i with approximate key <= threshold, in any order: every thread counts
    // its own, the wavefronts take their slots with one addition each; the largest such key
    int mine = 0;
    uint32_t my_max = 0u;
    for_keys<NK>(npt, [&](int e) {
        const uint32_t key = key_at(e);
        if (key <= thr_key) {   // the row's own token and padding carry 0xFFFFFFFF > thr_key
            ++mine;
            my_max = max(my_max, key);
        }
    });
    const int incl = wave_scan_i<OpSum>(mine, 0);
    my_max = (uint32_t)__builtin_amdgcn_readlane(wave_scan_i<OpMax>((int)(my_max ^ 0x80000000u), INT_MIN), 63) ^ 0x80000000u;
    int first = 0;
    if (lane == WAVE - 1) {
        first = atomicAdd(&sh.taken, incl);
        atomicMax(&sh.thr_max, my_max);
    }
    int slot = __builtin_amdgcn_readlane(first, WAVE - 1) + incl - mine;
    for_keys<NK>(npt, [&](int e) {   // slot < best <= CAP: the same keys as in the counting pass
        if (key_at(e) <= thr_key) sh.idx[slot++] = token_of(e);
    });
    __syncthreads();
    const int count = sh.taken;
    const float thr = ord_inv(sh.thr_max);   // every discarded token has an approximate key above this

    // The candidates in ascending order of (exact key, token).  Up to 1024 of them: buckets of equal
    // width over the keys' range (a monotone map, so buckets are in order), the candidates moved to
    // their buckets, and every candidate's rank is its bucket's start plus the number of smaller ones in
    // the bucket: a few elements each, five barriers in all, where a sorting network over 1024 takes
    // 55 steps and was half of this kernel's time (with the histogram above in place of the counting
    // passes, V = 16384, d = 8, k = 1000: 343 -> 188 us for the 16384 rows).  Rows with a crowded bucket
    // (many equal keys) take the network, and rows of more than 1024 candidates do.
    bool emitted = false;
    if (CAP <= 1024) {
        constexpr int CPT = CAP > TNT ? CAP / TNT : 1;
        double ck[CPT];
        int ct[CPT], at[CPT];
        float fmin_ = INFINITY, fmax_ = neg_inf_f();
        const double norm2 = (KEYS == KEYS_VECTORS || vecs) && metric != 0 ? own_norm2(own, d) : 0.0;
#pragma unroll
        for (int e = 0; e < CPT; ++e) {
            const int c = e * TNT + tid;
            if (c < count) {
                ct[e] = sh.idx[c];
                ck[e] = vecs == 0 && KEYS != KEYS_VECTORS ? exact_key<CT>(cb, d, i, ct[e], metric, vec4)
                        : metric == 0 ? exact_key_vec<CT, 0, 4>(cb, vecs, own, ct[e], 0.0)
                                      : exact_key_vec<CT, 1, 4>(cb, vecs, own, ct[e], norm2);
                fmin_ = fminf(fmin_, (float)ck[e]);
                fmax_ = fmaxf(fmax_, (float)ck[e]);
            }
        }
        fmin_ = -wave_max(-fmin_);
        fmax_ = wave_max(fmax_);
        if (lane == 0) { sh.red_u[wave] = __float_as_uint(fmin_); sh.red_u[TNW + wave] = __float_as_uint(fmax_); }
        __syncthreads();
        fmin_ = __uint_as_float(sh.red_u[0]);
        fmax_ = __uint_as_float(sh.red_u[TNW]);
#pragma unroll
        for (int w = 1; w < TNW; ++w) {
            fmin_ = fminf(fmin_, __uint_as_float(sh.red_u[w]));
            fmax_ = fmaxf(fmax_, __uint_as_float(sh.red_u[TNW + w]));
        }
        const float range = fmax_ - fmin_;   // no range (or none that floats can divide): one bucket
        const float scale = (range > 1e-30f && range < INFINITY) ? (float)(Shared::BUCKETS - 1) / range : 0.f;
        auto bucket_of = [&](double key) -> int {
            return scale > 0.f ? min((int)(((float)key - fmin_) * scale), Shared::BUCKETS - 1) : 0;
        };
#pragma unroll
        for (int e = 0; e < CPT; ++e)
            if (e * TNT + tid < count) at[e] = bucket_add(sh.hist, bucket_of(ck[e]));
        __syncthreads();
        bucket_starts<Shared::BUCKETS, TNT>(sh.hist, sh.red_c[1], tid, [&](int, int, int n) {
            if (n > CROWDED) sh.cut[2] = 1;
        });
        __syncthreads();
#pragma unroll
        for (int e = 0; e < CPT; ++e)
            if (e * TNT + tid < count) {
                const int p = bucket_start(sh.hist, bucket_of(ck[e])) + at[e];
                sh.key[p] = ck[e];
                sh.idx[p] = ct[e];
            }
        __syncthreads();
        if (!sh.cut[2]) {
            emitted = true;
            rank_in_buckets<Shared::BUCKETS, TNT, CAP>(sh, count, need, tid, bucket_of, orow);
        }
    }
    if (!emitted) {   // uniform
        if (CAP > 1024)
            for (int c = tid; c < count; c += TNT) sh.key[c] = exact_key<CT>(cb, d, i, sh.idx[c], metric, vec4);
        sort_candidates<TNT>(sh, count, need, tid, orow);
    }
    __syncthreads();
    // proof that no discarded token belongs to the row: every discarded j has an
    // approximate key above thr, hence an exact key above thr - err; the last
    // token taken must lie at or below that.
    bool ok = true;
    if (LIST || count < V - 1)
        ok = count >= need && proven(sh.last, thr, d, metric, err_rel, err_abs, err_norm, norms ? norms[i] : 0.f, *nmax, norms != nullptr);
    if (!ok && tid == 0) flags[row] = 1;
}

// ---- stage 2 for lists of tokens alone: every listed token's key in fp64, then as above ----
// Where a code is a few vectors the keys cost less than narrowing the list to the candidates wanted: no approximate
// keys are kept, and of the phases between which the workgroup waits (range, histogram, starts, boundary, compaction,
// range, histogram, starts, placing, ranking) four are left out.  One histogram over the list's exact keys finds
// the bucket in which the count passes `need`; the tokens up to it are placed and ranked as above.  If they are more than
// the LDS holds (many nearly equal keys), the keys below that bucket are set aside and the bucket itself is divided
// again, until they fit or its keys are equal; then the places come from a histogram of their own.
// Every token not on the list has a value below the row's threshold, which is what the proof uses.
// V = 16384, d = 8, k = 1000 (lists of 1672 tokens, 16384 rows): 172 us, and 182 for the selection from pairs, whose
// lists take the filtering contraction 80 us longer.
template <typename CT, int NP, int VECS, int METRIC>
__global__ __launch_bounds__(LIST_THREADS, 4) void knn_rank_list(const CT* cb, int V, int d, int k, int r0,
                                                                 FilterOut list, float err_rel, float err_abs,
                                                                 float err_norm, const float* norms, const float* nmax,
                                                                 const int* doubt, int32_t* out, int* flags) {
    constexpr int CAP = 1024, TNT = LIST_THREADS, TNW = TNT / WAVE;
    using Shared = SelectShared<CAP, TNT>;
    constexpr int BUCKETS = Shared::BUCKETS;
    __shared__ Shared sh;
    __shared__ float ends[2 * TNW];
    __shared__ double own[VECS * KeySum<CT, METRIC>::EPV];
    const int row = blockIdx.x;
    const int i = r0 + row;
    const int tid = threadIdx.x;
    const int lane = tid & (WAVE - 1);
    const int wave = tid >> 6;
    int32_t* orow = out + (int64_t)i * k;
    const int need = k - 1;                                 // at least one: the plan wants more than 64
    const int want = min(V - 1, need + 8 + need / 128);
    const int listed = list.counts[row];
    if (tid == 0) {
        orow[0] = i;
        flags[row] = 0;
        sh.cut[2] = 0;
        sh.last = INFINITY;
    }
    if (listed > min(list.cap, NP * TNT) || listed < want || (METRIC != 0 && *doubt)) {
        if (tid == 0) flags[row] = 1;
        return;
    }
    int tok[NP];
    double key[NP];
    {
        const uint32_t* lrow = static_cast<const uint32_t*>(list.cand) + (int64_t)row * list.cap;
#pragma unroll
        for (int e = 0; e < NP; ++e) tok[e] = (int)lrow[min(e * TNT + tid, listed - 1)];   // no branch: all loads in flight together
    }
    own_code<CT>(cb + (int64_t)i * d, d, own, tid, TNT);
    for (int w = tid; w < BUCKETS / 2; w += TNT) sh.hist[w] = 0u;
    __syncthreads();
    const double norm2 = METRIC != 0 ? own_norm2(own, d) : 0.0;
    float low = INFINITY, high = neg_inf_f();
    constexpr int BATCH = VECS > 1 ? 2 : 4;                 // slots whose codes are on their way together
#pragma unroll
    for (int e0 = 0; e0 < NP; e0 += BATCH)
        if (e0 * TNT < listed) {                            // uniform
            vec4u v[BATCH][VECS];
#pragma unroll
            for (int u = 0; u < BATCH; ++u)
#pragma unroll
                for (int q = 0; q < VECS; ++q) v[u][q] = reinterpret_cast<const vec4u*>(cb)[(uint32_t)tok[e0 + u] * VECS + q];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                KeySum<CT, METRIC> sum;
#pragma unroll
                for (int q = 0; q < VECS; ++q) sum.add(v[u][q], own + q * KeySum<CT, METRIC>::EPV);
                key[e0 + u] = sum.key(norm2);
                if ((e0 + u) * TNT + tid < listed) {
                    low = fminf(low, (float)key[e0 + u]);
                    high = fmaxf(high, (float)key[e0 + u]);
                }
            }
        }
    // `in`: keys that certainly belong to the first ones, `open`: those the next histogram is over
    uint32_t in = 0, open = 0;
#pragma unroll
    for (int e = 0; e < NP; ++e) open |= e * TNT + tid < listed ? 1u << e : 0u;
    int at[NP];                           // bucket * 65536 + place in it
    float scale = 0.f;
    auto bucket_of = [&](double x) -> int {   // keys a rounding outside the range belong to its ends
        return scale > 0.f ? min(max((int)(((float)x - low) * scale), 0), BUCKETS - 1) : 0;
    };
    // range of the keys of `mask` (low, high as this thread has them), their histogram, its starts
    auto histogram = [&](uint32_t mask, auto each) {
        low = -wave_max(-low);
        high = wave_max(high);
        if (lane == 0) {
            ends[wave] = low;
            ends[TNW + wave] = high;
        }
        __syncthreads();
        low = ends[0];
        high = ends[TNW];
#pragma unroll
        for (int w = 1; w < TNW; ++w) {
            low = fminf(low, ends[w]);
            high = fmaxf(high, ends[TNW + w]);
        }
        // No range, or none that floats can divide: one bucket.  Codes of small coordinates have small ranges (2047 divided
        // by the least one here is 0.6 of the largest float).
        const float range = high - low;
        scale = (range > 1e-35f && range < INFINITY) ? (float)(BUCKETS - 1) / range : 0.f;
#pragma unroll
        for (int e = 0; e < NP; ++e)
            if ((mask >> e) & 1u) {
                const int b = bucket_of(key[e]);
                at[e] = (b << 16) + bucket_add(sh.hist, b);
            }
        __syncthreads();
        bucket_starts<BUCKETS, TNT>(sh.hist, sh.red_c[0], tid, each);
        __syncthreads();
    };
    auto clear = [&] {
        __syncthreads();
        for (int w = tid; w < BUCKETS / 2; w += TNT) sh.hist[w] = 0u;
        __syncthreads();
    };
    int base = 0;                         // keys set aside so far
    auto find_cut = [&](int bucket, int start, int n) {
        if (base + start < need && base + start + n >= need) {
            sh.cut[0] = bucket;
            sh.cut[1] = start + n;
            sh.red_u[0] = (unsigned)start;
        }
        if (n > CROWDED && base + start < need) sh.cut[2] = 1;
    };
    histogram(open, find_cut);
    int count = sh.cut[1];
    if (count > CAP) {                    // uniform
        for (int round = 0; round < 16 && base + count > CAP; ++round) {
            const int cut = sh.cut[0], below = (int)sh.red_u[0];
            if (scale == 0.f) break;      // as many equal keys as that
            const uint32_t was = open;
            open = 0;
            float l = INFINITY, h = neg_inf_f();
#pragma unroll
            for (int e = 0; e < NP; ++e)
                if ((was >> e) & 1u) {
                    const int b = at[e] >> 16;
                    if (b < cut) in |= 1u << e;
                    else if (b == cut) {
                        open |= 1u << e;
                        l = fminf(l, (float)key[e]);
                        h = fmaxf(h, (float)key[e]);
                    }
                }
            base += below;
            low = l;
            high = h;
            clear();
            histogram(open, find_cut);
            count = sh.cut[1];
        }
        if (base + count > CAP) {         // uniform: the all-pairs pass
            if (tid == 0) flags[row] = 1;
            return;
        }
        const int cut = sh.cut[0];
        float l = INFINITY, h = neg_inf_f();
#pragma unroll
        for (int e = 0; e < NP; ++e) {
            if (((open >> e) & 1u) && (at[e] >> 16) <= cut) in |= 1u << e;
            if ((in >> e) & 1u) {
                l = fminf(l, (float)key[e]);
                h = fmaxf(h, (float)key[e]);
            }
        }
        count += base;
        low = l;
        high = h;
        clear();
        if (tid == 0) sh.cut[2] = 0;
        histogram(in, [&](int, int, int n) {
            if (n > CROWDED) sh.cut[2] = 1;
        });
    } else {
        const int limit = (sh.cut[0] + 1) << 16;
#pragma unroll
        for (int e = 0; e < NP; ++e)
            if (((open >> e) & 1u) && at[e] < limit) in |= 1u << e;
    }
    // `count` keys, in their buckets
#pragma unroll
    for (int e = 0; e < NP; ++e)
        if ((in >> e) & 1u) {
            const int p = bucket_start(sh.hist, at[e] >> 16) + (at[e] & 0xFFFF);
            sh.key[p] = key[e];
            sh.idx[p] = tok[e];
        }
    __syncthreads();
    if (!sh.cut[2]) rank_in_buckets<BUCKETS, TNT, CAP>(sh, count, need, tid, bucket_of, orow);
    else sort_candidates<TNT>(sh, count, need, tid, orow);
    __syncthreads();
    // proof that no token left out belongs to the row: its value is below the threshold
    const float thr = key_of_value<METRIC>(list.thr[row], norms[i]);
    const bool ok = proven(sh.last, thr, d, METRIC, err_rel, err_abs, err_norm, METRIC == 0 ? norms[i] : 0.f, *nmax, METRIC == 0);
    if (tid == 0 && !ok) flags[row] = 1;
}

// ---- stage 3: flagged rows, all V keys in fp64, rank by counting ----
template <typename CT>
__global__ __launch_bounds__(NT) void knn_exact_rows(const CT* cb, int V, int d, int k, int metric,
                                                     const int* flags, double* bufs, int32_t* out, int* stats) {
    const int tid = threadIdx.x;
    double* buf = bufs + (int64_t)blockIdx.x * V;
    const int need = k - 1;
    // the workgroup's rows are blockIdx.x, blockIdx.x + gridDim.x, ...: all their flags are looked at
    // at once first, and a workgroup with none set is done
    int any = 0;
    for (int row = blockIdx.x + tid * gridDim.x; row < V; row += NT * gridDim.x) any |= flags[row];
    if (!__syncthreads_or(any)) return;
    for (int i = blockIdx.x; i < V; i += gridDim.x) {
        if (!flags[i]) continue;  // uniform
        if (tid == 0) atomicAdd(stats, 1);
        __syncthreads();
        for (int j = tid; j < V; j += NT)
            buf[j] = (j == i) ? NAN : exact_key<CT>(cb, d, i, j, metric, false);   // NaN: counted by no comparison below
        __threadfence_block();
        __syncthreads();
        int32_t* orow = out + (int64_t)i * k;
        for (int j = tid; j < V; j += NT) {
            if (j == i) continue;
            const double kj = buf[j];
            int rank = 0;
            for (int o = 0; o < V; ++o) {
                const double ko = buf[o];
                rank += (ko < kj || (ko == kj && o < j)) ? 1 : 0;
            }
            if (rank < need) orow[1 + rank] = j;
        }
    }
}

__global__ void knn_clear_stats(int* stats, float* nmax, int* doubt) {
    stats[threadIdx.x] = 0;
    if (threadIdx.x == 0) {
        *nmax = 0.f;
        doubt[0] = doubt[1] = 0;
    }
}
__global__ void knn_copy_stats(const int* stats, int32_t* out) { *out = stats[0]; }

template <typename CT>
static hipError_t build_typed(const KnnArgs& a, const KnnLayout& L, hipStream_t stream) {
    unsigned char* ws = static_cast<unsigned char*>(a.workspace);
    float* dist = reinterpret_cast<float*>(ws + L.dist);
    int* flags = reinterpret_cast<int*>(ws + L.flags);
    double* slow = reinterpret_cast<double*>(ws + L.slow);
    const CT* cb = static_cast<const CT*>(a.codebook);
    int* stats = reinterpret_cast<int*>(ws + L.stats);
    float* norms = reinterpret_cast<float*>(ws + L.norms);
    float* nmax = reinterpret_cast<float*>(ws + L.nmax);
    int* doubt = reinterpret_cast<int*>(nmax) + 1;   // a code whose cosine keys the error bound does not cover; one not plain
    hipLaunchKernelGGL(knn_clear_stats, dim3(1), dim3(64), 0, stream, stats, nmax, doubt);
    // matrix-core path: rows 16-byte aligned and coordinates in whole vectors
    const bool aligned = (reinterpret_cast<uintptr_t>(a.codebook) & 15) == 0;
    const bool mfma = aligned && (sizeof(CT) == 2 ? (a.d % 8) == 0 : (a.d % 4) == 0) && a.V >= 32;
    const FilterPlan& plan = L.filter;   // the caller lays the filtering path out only for an aligned codebook
    // one rounding is at most 2^-23 relative here (twice the fp32 unit, to cover a
    // contraction that truncates); a d-term sum takes d + 8 of them
    const float gamma = (float)(a.d + 8) * 1.1920929e-7f;
    float err_rel, err_abs, err_norm;
    if (mfma) {
        const int per_wg = a.d * (int)sizeof(CT) / 16 >= NORM_WAVE_VECS ? NORM_ROWS : NT;
        hipLaunchKernelGGL((knn_norms<CT>), dim3((a.V + per_wg - 1) / per_wg), dim3(NT), 0, stream, cb, a.V, a.d,
                           a.metric, norms, nmax, doubt);
        // n_i + n_j - 2 G: errors of the two norms and of G are each below gamma (n_i + n_j) / 2 ... gamma (n_i + n_j)
        err_rel = 0.f;
        err_abs = a.metric == 0 ? 0.f : 4.f * gamma;
        err_norm = a.metric == 0 ? 2.f * gamma : 0.f;
    } else {
        // direct evaluation: relative to the key for squared l2 (a sum of squares);
        // absolute, against |cos| <= 1, for the cosine key
        err_rel = a.metric == 0 ? gamma : 0.f;
        err_abs = a.metric == 0 ? 0.f : 2.f * gamma;
        err_norm = 0.f;
    }
    uint4* packed = reinterpret_cast<uint4*>(ws + L.packed);
    uint4* spacked = reinterpret_cast<uint4*>(ws + L.spacked);
    float* fold = reinterpret_cast<float*>(ws + L.fold);
    const int steps = (int)packed_steps(a.d, sizeof(CT) == 2 ? 1 : 0);
    float* sfold = reinterpret_cast<float*>(ws + L.sfold);
    float* snorms = reinterpret_cast<float*>(ws + L.snorms);
    float* skeys = reinterpret_cast<float*>(ws + L.skeys);
    FilterOut fo;
    fo.thr = reinterpret_cast<float*>(ws + L.thr);
    fo.counts = reinterpret_cast<int*>(ws + L.counts);
    fo.cand = ws + L.cand;
    fo.cap = plan.cap;
    const FilterOut no_list = {nullptr, nullptr, nullptr, 0};
    if (plan.use) {
        if (!mfma) return hipErrorInvalidValue;
        // v = G - n_j / 2 is one sum of d + 1 terms: its error, doubled, is below gamma (n_i + 2 n_j), and the
        // two norms' add gamma (n_i + n_j)
        if (a.metric == 0) err_norm = 3.f * gamma;
        const int64_t threads = (int64_t)(packed_tiles(a.V) + packed_tiles(plan.S)) * steps * WAVE;
        const dim3 grid((unsigned)((threads + NT - 1) / NT));
        if (a.metric == 0)
            hipLaunchKernelGGL((knn_pack<CT, 0>), grid, dim3(NT), 0, stream, cb, norms, a.V, a.d, plan.S, steps, packed,
                               spacked, fold, sfold, snorms);
        else
            hipLaunchKernelGGL((knn_pack<CT, 1>), grid, dim3(NT), 0, stream, cb, norms, a.V, a.d, plan.S, steps, packed,
                               spacked, fold, sfold, snorms);
    }
    const int vecs = mfma ? a.d * (int)sizeof(CT) / 16 : 0;   // rows of whole vectors at aligned addresses
    const int key_vecs = a.d <= VEC_MAX_D ? vecs : 0;
    // The exact keys of a selection from whole rows read codes of up to 32 bytes by elements where 256 slots do and a thread holds 32
    // keys or more (with fewer there is no difference), of 64 bytes as well unless many cosine keys each take the own code's norm.
    // Vectors / elements, fp32: V = 8192, k = 30, cosine, d = 8 204.5 / 201.6 us, d = 16 219.3 / 216.7; V = 4000, d = 16, k = 200, l2 82.3 /
    // 82.1, cosine 96.9 / 106.7; V = 4000, d = 32, k = 200, l2 94.5 / 95.4.
    const int want_slots = candidate_slots(a.k);
    auto row_vecs = [&](int keys, int slots) {
        return key_vecs > (slots > 256 || keys == 8 ? 0 : a.metric == 0 || want_slots <= 128 ? 4 : 2);
    };
    auto filter = [&](int r0, int rows) {
        const int nrt = (rows + 127) / 128;
#define LANTERN_LAUNCH_FILTER(METRICV, FORMV, TTV)                                                                       \
        hipLaunchKernelGGL((knn_filter_list<CT, METRICV, FORMV, TTV>),                                                   \
                           dim3((unsigned)((nrt + 7) / 8 * 8 * ((a.V + 128 * TTV - 1) / (128 * TTV)))), dim3(NT), 0, stream, \
                           packed, fold, norms, a.V, steps, r0, rows, doubt, fo)
        if (plan.tokens && plan.wide_tiles) {
            if (a.metric == 0) LANTERN_LAUNCH_FILTER(0, LIST_TOKENS, 4);
            else LANTERN_LAUNCH_FILTER(1, LIST_TOKENS, 4);
        } else if (plan.tokens) {
            if (a.metric == 0) LANTERN_LAUNCH_FILTER(0, LIST_TOKENS, 1);
            else LANTERN_LAUNCH_FILTER(1, LIST_TOKENS, 1);
        } else if (a.metric == 0) LANTERN_LAUNCH_FILTER(0, LIST_PAIRS, 1);
        else LANTERN_LAUNCH_FILTER(1, LIST_PAIRS, 1);
#undef LANTERN_LAUNCH_FILTER
    };
    // thresholds of a block of rows from the sample
    auto thresholds = [&](int r0, int rows) {
        float* least = const_cast<float*>(fo.thr);
        if (plan.S > THRESHOLDS_MAX_S) {
            hipLaunchKernelGGL((knn_sample_keys<CT>), dim3((plan.S + 127) / 128, (rows + 127) / 128), dim3(NT), 0, stream,
                               packed, spacked, norms, snorms, a.V, plan.S, steps, r0, rows, a.metric, skeys);
            hipLaunchKernelGGL(knn_sample_rank, dim3((rows + NW - 1) / NW), dim3(NT), 0, stream, skeys, plan.S, rows,
                               plan.rank, plan.slack, norms, r0, a.metric, least, fo.counts);
            return;
        }
        const double share = (plan.rank + 0.5 * plan.slack) / plan.S;
        const double z = normal_upper_quantile(share);
        const float per_count = (float)(1.0 / (plan.S * normal_density(z)));
#define LANTERN_LAUNCH_THRESHOLDS(METRICV, TPWV)                                                                         \
        hipLaunchKernelGGL((knn_thresholds<CT, METRICV, TPWV>), dim3((rows + 31) / 32), dim3(THR_THREADS), 0, stream, packed, \
                           spacked, sfold, a.V, plan.S, steps, r0, rows, plan.rank, plan.slack, (float)z, per_count, doubt, least, \
                           fo.counts)
#define LANTERN_LAUNCH_THRESHOLDS_TPW(METRICV)                                                                           \
        do {                                                                                                             \
            if (plan.S <= 512) LANTERN_LAUNCH_THRESHOLDS(METRICV, 1);                                                    \
            else if (plan.S <= 1024) LANTERN_LAUNCH_THRESHOLDS(METRICV, 2);                                              \
            else LANTERN_LAUNCH_THRESHOLDS(METRICV, 4);                                                                  \
        } while (0)
        if (a.metric == 0) LANTERN_LAUNCH_THRESHOLDS_TPW(0);
        else LANTERN_LAUNCH_THRESHOLDS_TPW(1);
#undef LANTERN_LAUNCH_THRESHOLDS_TPW
#undef LANTERN_LAUNCH_THRESHOLDS
    };
    for (int r0 = 0; r0 < a.V; r0 += L.row_block) {
        const int rows = (a.V - r0) < L.row_block ? (a.V - r0) : L.row_block;
        const float* nsel = mfma && a.metric == 0 ? norms : nullptr;
        // candidate capacity: the smallest of 256 / 1024 / 2048 / 4096 slots that holds k-1+pad.  The
        // selection is bound by the latency of its many short phases, so its throughput is the number
        // of workgroups a compute unit holds at once, and that number is set by this LDS footprint
        // (12 bytes a slot).
#define LANTERN_LAUNCH_SELECT_KEYS(NKV, CAPV, TNTV, LISTV, KEYSV, VECSV)                                    \
        hipLaunchKernelGGL((knn_select<CT, NKV, CAPV, TNTV, LISTV, KEYSV>), dim3(rows), dim3(TNTV),         \
                           own_code_bytes(a.d, VECSV), stream, cb,                                          \
                           a.V, a.d, a.k, a.metric, r0, dist, LISTV ? fo : no_list, err_rel, err_abs,       \
                           err_norm, nsel, nmax, doubt, a.out, flags + r0, VECSV)
        // whole rows of keys; beyond 1024 candidates their exact keys are taken by elements
#define LANTERN_LAUNCH_SELECT_ROWS(NKV, CAPV, TNTV)                                                         \
        do {                                                                                                \
            /* of 1024 slots a kernel of both forms spills less than one of vectors alone, but for these two */ \
            constexpr bool BOTH = (CAPV) == 1024 && (sizeof(CT) == 2 ? NKV != 32 : NKV != 8);               \
            constexpr int BY_VECTORS = (CAPV) > 1024 ? KEYS_ELEMENTS : BOTH ? KEYS_EITHER : KEYS_VECTORS;   \
            if ((CAPV) > 1024 || !row_vecs(NKV, CAPV)) LANTERN_LAUNCH_SELECT_KEYS(NKV, CAPV, TNTV, false, KEYS_ELEMENTS, 0); \
            else LANTERN_LAUNCH_SELECT_KEYS(NKV, CAPV, TNTV, false, BY_VECTORS, key_vecs);                  \
        } while (0)
#define LANTERN_LAUNCH_SELECT_LIST(NKV, CAPV, TNTV) LANTERN_LAUNCH_SELECT_KEYS(NKV, CAPV, TNTV, true, KEYS_EITHER, key_vecs)
        if (plan.use) {
            // thresholds from the sample, then the contraction that keeps what lies below them
            thresholds(r0, rows);
            filter(r0, rows);
            static_assert(LIST_THREADS == NT, "threads per row of the selection from lists");
            const int pairs = plan_pairs(plan, a.k);   // 64 < want_slots <= 1024
#define LANTERN_LAUNCH_RANK(NPV)                                                                                         \
            do {                                                                                                         \
                auto* kernel = a.metric == 0 ? (vecs == 1   ? &knn_rank_list<CT, NPV, 1, 0>                              \
                                                : vecs == 2 ? &knn_rank_list<CT, NPV, 2, 0>                              \
                                                            : &knn_rank_list<CT, NPV, 4, 0>)                             \
                                             : (vecs == 1   ? &knn_rank_list<CT, NPV, 1, 1>                              \
                                                : vecs == 2 ? &knn_rank_list<CT, NPV, 2, 1>                              \
                                                            : &knn_rank_list<CT, NPV, 4, 1>);                            \
                hipLaunchKernelGGL(kernel, dim3(rows), dim3(LIST_THREADS), 0, stream, cb, a.V, a.d, a.k, r0, fo, err_rel, \
                                   err_abs, err_norm, norms, nmax, doubt, a.out, flags + r0);                            \
            } while (0)
            if (plan.tokens) {
                if (pairs == 8) LANTERN_LAUNCH_RANK(8);
                else if (pairs == 12) LANTERN_LAUNCH_RANK(12);
                else LANTERN_LAUNCH_RANK(16);
#undef LANTERN_LAUNCH_RANK
            } else if (want_slots <= 256) {
                // two wavefronts a row: its candidates would leave some of four without any
                static_assert(LIST_THREADS == 2 * NARROW_THREADS, "twice the pairs per thread");
                if (pairs == 4) LANTERN_LAUNCH_SELECT_LIST(8, 256, NARROW_THREADS);
                else if (pairs == 8) LANTERN_LAUNCH_SELECT_LIST(16, 256, NARROW_THREADS);
                else if (pairs == 12) LANTERN_LAUNCH_SELECT_LIST(24, 256, NARROW_THREADS);
                else LANTERN_LAUNCH_SELECT_LIST(32, 256, NARROW_THREADS);
            } else if (pairs == 8) LANTERN_LAUNCH_SELECT_LIST(8, 1024, NT);
            else if (pairs == 12) LANTERN_LAUNCH_SELECT_LIST(12, 1024, NT);
            else LANTERN_LAUNCH_SELECT_LIST(16, 1024, NT);
        } else {
            if (mfma)
                hipLaunchKernelGGL((knn_dist_mfma<CT>), dim3((a.V + 127) / 128, (rows + 127) / 128), dim3(NT), 0, stream,
                                   cb, norms, a.V, a.d, r0, rows, a.metric, dist);
            else
                hipLaunchKernelGGL((knn_dist_direct<CT>), dim3((a.V + NT - 1) / NT, rows), dim3(NT), 0, stream,
                                   cb, a.V, a.d, r0, a.metric, dist, doubt);
#define LANTERN_LAUNCH_SELECT_NK(NKV, TNTV)                                                                 \
            do {                                                                                            \
                if (want_slots <= 256) LANTERN_LAUNCH_SELECT_ROWS(NKV, 256, TNTV);                        \
                else if (want_slots <= 1024) LANTERN_LAUNCH_SELECT_ROWS(NKV, 1024, TNTV);                 \
                else if (want_slots <= 2048) LANTERN_LAUNCH_SELECT_ROWS(NKV, 2048, TNTV);                 \
                else LANTERN_LAUNCH_SELECT_ROWS(NKV, CAND_CAP, TNTV);                                     \
            } while (0)
            // threads per row and keys per thread: up to 64 keys per thread in registers; vocabularies
            // beyond 64 x 256 tokens take 512 threads per row (32 keys per thread on 512 threads measured
            // the same as 64 on 256 at V = 16384); beyond 64 x 512 the keys are re-read in every pass
            if (a.V <= 8 * NT) LANTERN_LAUNCH_SELECT_NK(8, NT);
            else if (a.V <= 32 * NT) LANTERN_LAUNCH_SELECT_NK(32, NT);
            else if (a.V <= 64 * NT) LANTERN_LAUNCH_SELECT_NK(64, NT);
            else if (a.V <= 64 * 512) LANTERN_LAUNCH_SELECT_NK(64, 512);
            else LANTERN_LAUNCH_SELECT_NK(0, NT);
#undef LANTERN_LAUNCH_SELECT_NK
        }
#undef LANTERN_LAUNCH_SELECT_ROWS
#undef LANTERN_LAUNCH_SELECT_LIST
#undef LANTERN_LAUNCH_SELECT_KEYS
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // flagged rows of the whole table
    const int wgs = a.V < L.slow_wgs ? a.V : L.slow_wgs;
    hipLaunchKernelGGL((knn_exact_rows<CT>), dim3(wgs), dim3(NT), 0, stream, cb, a.V, a.d, a.k, a.metric, flags,
                       slow, a.out, stats);
    return hipGetLastError();
}

hipError_t launch_build_knn(const KnnArgs& a, hipStream_t stream) {
    // A codebook that is not 16-byte aligned cannot take the filtering path: it gets whole key blocks, for which
    // the workspace has room as well.
    const FilterPlan plan = filter_plan(a.V, a.d, a.k, a.cb_dtype);
    KnnLayout L = knn_layout(a.V, a.d, a.cb_dtype, plan, plan.use ? FILTER_ROW_BLOCK : whole_row_block(a.V), SLOW_WGS);
    if (plan.use && (reinterpret_cast<uintptr_t>(a.codebook) & 15) != 0)
        L = knn_layout(a.V, a.d, a.cb_dtype, NO_FILTER, whole_row_block(a.V), SLOW_WGS);
    if (a.cb_dtype == 0) return build_typed<float>(a, L, stream);
    return build_typed<uint16_t>(a, L, stream);
}

// The same build with the library's static scratch as workspace; a.workspace is ignored.
// exact_rows: device int32 that receives the number of rows ranked by the all-pairs pass, or null.
hipError_t launch_build_knn_static(const KnnArgs& a_in, int32_t* exact_rows, hipStream_t stream) {
    const KnnLayout L = knn_layout_static(a_in.V, a_in.d, a_in.cb_dtype);
    if (L.row_block == 0) return hipErrorInvalidValue;   // the host entry has checked this
    KnnArgs a = a_in;
    hipError_t e = static_scratch_ptr(&a.workspace);
    if (e != hipSuccess) return e;
    e = a.cb_dtype == 0 ? build_typed<float>(a, L, stream) : build_typed<uint16_t>(a, L, stream);
    if (e != hipSuccess) return e;
    if (exact_rows) {
        hipLaunchKernelGGL(knn_copy_stats, dim3(1), dim3(1), 0, stream,
                           reinterpret_cast<const int*>(static_cast<unsigned char*>(a.workspace) + L.stats), exact_rows);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace lantern

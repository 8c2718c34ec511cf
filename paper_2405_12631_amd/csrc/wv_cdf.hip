// Discretised mixture (Gaussian or Laplacian components) -> 16-bit integer CDF tables.
//
// Row n (one coefficient) has N_s + 1 entries cdf[j] = j + F_j with
// F_j = floor(F_max * C_j), C_j the normalised mixture CDF at the boundary
// sym_min + j - 0.5, F_max = 2^16 - N_s; entry N_s (= 2^16) is stored as 0.
// The exact value of the floor is produced:
//   * outside [j_lo, j_hi], where every component is at least TZ scales away
//     from the boundary (TZ = 4.5 Gaussian, 11 Laplace), the value is known
//     without evaluating Phi: C_j <= Phi(-TZ) < 1/F_max gives F_j = 0 below,
//     and 0 < 1 - C_j < 1/F_max gives F_j = F_max - 1 above;
//   * inside, the lower tail sum is used when C_j <= 1/2, else the upper tail
//     (F_j = F_max - ceil(F_max * (1 - C_j)), at least one count below F_max),
//     so no digits are lost to 1 - tiny rounding to 1;
//   * a running maximum makes the row non-decreasing.
// What bounds it: outside the rows' windows only the writes (260 bytes a row), inside them the
// tails, about 50 vector instructions per component and entry.  Windows differ: for scales spread
// over a decade their mean is 25 entries, but the longest of 64 rows has 101.  So a workgroup
// fills its rows' entries outside the windows in LDS, deals all the window entries evenly to its
// threads (a prefix sum of the window lengths, a binary search per entry), and copies the rows out
// as one block.  (One thread or four lanes per row, as before, step through the longest window of a
// wave: 2.4 M such rows 1239 us, 1152 rows 27 us; now 335 us and 5 us.  For rows as narrow as an
// untrained model's, ten entries each, the search and the fill cost as much as the even deal saves: a
// batch of 8 Mpixels 2.25 and 2.26 ms, one of 51 Mpixels 9.6 before and 11.0 now, 4.1 TB/s.  128 or 512
// threads, or 32 rows, 11.3 to 13.8.)  The running maximum is the identity up to rounding, so entries are
// only compared with their predecessors, and a row is gone through again if one of them is larger.
#include "wv_device.h"
#include "wv_internal.h"

#include <mutex>

namespace wv {
namespace {

constexpr int NT = 256;     // threads
constexpr int MAXE = 256;   // max entries per row (N_s + 1)

template <int K, int DIST, int ROWS>
__global__ __launch_bounds__(NT) void cdf_k(const float* __restrict__ params, long long n, int smin, int nsym,
                                           uint16_t* __restrict__ out) {
    extern __shared__ __attribute__((aligned(16))) uint16_t tab[];   // [ROWS][nsym + 1]
    __shared__ CdfRow<K, DIST> R[ROWS];
    __shared__ int win[ROWS][2];        // evaluated entries j1 <= j < j2
    __shared__ int first[ROWS + 1];     // of a row's entries among the workgroup's
    __shared__ int bad[ROWS], anybad;   // rows whose F decreases somewhere
    const int tid = threadIdx.x, lane = tid & 63;
    const int E = nsym + 1;
    const long long row0 = (long long)blockIdx.x * ROWS;
    const int nrows = (int)((n - row0) < ROWS ? (n - row0) : ROWS);
    if (tid < 64) {
        int len = 0;
        if (tid < ROWS) {
            CdfRow<K, DIST> r;
            int j1 = 1, j2 = 1;
            if (tid < nrows) {
                cdf_setup<K, DIST>(params + (row0 + tid) * (3 * K), smin, nsym, r);
                R[tid] = r;
                j1 = min(max(r.jlo, 1), nsym);
                j2 = max(min(r.jhi + 1, nsym), j1);
            }
            win[tid][0] = j1;
            win[tid][1] = j2;
            bad[tid] = 0;
            len = j2 - j1;
        }
        int sum = len;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_up(sum, d);
            if (lane >= d) sum += o;
        }
        if (tid < ROWS) first[tid + 1] = sum;
        if (tid == 0) first[0] = anybad = 0;
    }
    __syncthreads();
    const int Fmax = 65536 - nsym;
    {   // cdf[j] = j below the window, j + F_max - 1 above it; the last entry 0 (a thread keeps its row)
        const int r = tid % ROWS, j2 = win[r][1];
        if ((E & 1) == 0) {
            uint32_t* w = reinterpret_cast<uint32_t*>(tab + r * E);
            for (int q = tid / ROWS; q < E / 2; q += NT / ROWS) {
                const int j = 2 * q;
                const uint32_t a = j + (j >= j2 ? Fmax - 1 : 0), b = j + 1 + (j + 1 >= j2 ? Fmax - 1 : 0);
                w[q] = (a & 0xffffu) | (j + 1 == nsym ? 0u : b << 16);
            }
        } else {
            for (int j = tid / ROWS; j < E; j += NT / ROWS)
                tab[r * E + j] = j == nsym ? (uint16_t)0 : (uint16_t)(j + (j >= j2 ? Fmax - 1 : 0));
        }
    }
    __syncthreads();
    const int total = first[ROWS];
    for (int e0 = tid - lane; e0 < total; e0 += NT) {
        const int e = min(e0 + lane, total - 1);
        int r = 0;
#pragma unroll
        for (int d = ROWS / 2; d >= 1; d >>= 1)   // last row with first[r] <= e
            if (first[r + d] <= e) r += d;
        const int f = first[r], j1 = win[r][0], j = j1 + e - f;
        const CdfRow<K, DIST> row = R[r];
        const int F = max(cdf_F_in<K, DIST>(row, j), 0);
        tab[r * E + j] = (uint16_t)(j + F);
        // the row's entry before this one, except for the first lane (checked below)
        const int before = __builtin_amdgcn_update_dpp(0, F, 0x138, 0xf, 0xf, false);   // wave_shr:1
        if (lane > 0 && e > f && F < before) bad[r] = anybad = 1;
    }
    __syncthreads();
    for (int e = 64 * tid; e < total; e += 64 * NT) {   // entries that a first lane evaluated
        int r = 0;
#pragma unroll
        for (int d = ROWS / 2; d >= 1; d >>= 1)
            if (first[r + d] <= e) r += d;
        const uint16_t* c = tab + r * E + win[r][0] + e - first[r];
        if (e > first[r] && c[0] <= c[-1]) bad[r] = anybad = 1;
    }
    __syncthreads();
    if (anybad) {
        if (tid < ROWS && bad[tid]) {   // running maximum of F
            int m = 0;
            for (int j = win[tid][0]; j < nsym; ++j) {
                m = max(m, (int)tab[tid * E + j] - j);
                tab[tid * E + j] = (uint16_t)(j + m);
            }
        }
        __syncthreads();
    }
    // Contiguous copy of this block's rows.
    uint16_t* dst = out + row0 * E;
    const int nel = nrows * E;
    if ((((uintptr_t)dst) & 15) == 0 && (nel & 7) == 0) {
        const uint4* src4 = reinterpret_cast<const uint4*>(tab);
        uint4* dst4 = reinterpret_cast<uint4*>(dst);
        for (int i = tid; i < nel / 8; i += NT) dst4[i] = src4[i];
    } else {
        for (int i = tid; i < nel; i += NT) dst[i] = tab[i];
    }
}

}  // namespace

hipError_t launch_cdf(const float* params, long long n, int K, int dist, int smin, int nsym,
                      uint16_t* cdf, hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (nsym + 1 > MAXE || nsym < 2) return hipErrorInvalidValue;
    // 64 rows per workgroup share the fixed work best; up to about 100 000 rows (1500 such workgroups,
    // six per CU) 16 rows finish sooner: 1152 rows 5.1 against 9.4 us, 74 000 rows 18.0 against
    // 18.8 us, 150 000 rows 30.4 against 28.8 us.
    const bool small = n <= 96 * 1024;
    const int rows = small ? 16 : 64;
    const unsigned g = (unsigned)((n + rows - 1) / rows);
    const size_t lds = ((size_t)rows * (nsym + 1) * sizeof(uint16_t) + 15) & ~(size_t)15;
#define WV_CDF_CASE(KK, DD)                                                                                     \
    if (K == KK && dist == DD) {                                                                                \
        if (small)                                                                                              \
            hipLaunchKernelGGL((cdf_k<KK, DD, 16>), dim3(g), dim3(NT), lds, s, params, n, smin, nsym, cdf);        \
        else                                                                                                    \
            hipLaunchKernelGGL((cdf_k<KK, DD, 64>), dim3(g), dim3(NT), lds, s, params, n, smin, nsym, cdf);        \
        return hipGetLastError();                                                                               \
    }
    WV_CDF_CASE(1, 0) WV_CDF_CASE(2, 0) WV_CDF_CASE(3, 0) WV_CDF_CASE(4, 0)
    WV_CDF_CASE(1, 1) WV_CDF_CASE(2, 1) WV_CDF_CASE(3, 1) WV_CDF_CASE(4, 1)
#undef WV_CDF_CASE
    return hipErrorInvalidValue;
}


// ---- lossless trim of CDF rows (for the copy to the host coder) ----------
// In a row, F_j = cdf[j] - j (j = 1 .. nsym-1) is non-decreasing, 0 below the
// mass window and F_max - 1 above it (F_max = 2^16 - nsym; the upper tail keeps
// at least one count, so F never reaches F_max).  The row is therefore fixed by
// lo = 1 + #{F_j = 0}, len = #{0 < F_j < F_max - 1} and F_lo .. F_{lo+len-1};
// both counts come from binary searches.  Rows go 256 to a block: the first kernel
// writes (lo, len) and the block's sum of len, the second scans the block sums,
// the third writes each row's F values at its offset.
namespace {

__global__ __launch_bounds__(256) void trim_len_k(const uint16_t* __restrict__ cdf, long long n, int nsym,
                                                  uint8_t* __restrict__ lolen, long long* __restrict__ bsum) {
    __shared__ int red[256];
    const long long row = (long long)blockIdx.x * 256 + threadIdx.x;
    int len = 0;
    if (row < n) {
        const uint16_t* r = cdf + row * (nsym + 1);
        const int ftop = 65536 - nsym - 1;   // F_max - 1
        // first j in [1, nsym) with F_j > 0 (nsym if none)
        int a = 1, b = nsym;
        while (a < b) {
            const int mid = (a + b) >> 1;
            if ((int)r[mid] - mid > 0) b = mid; else a = mid + 1;
        }
        const int lo = a;
        // first j in [lo, nsym) with F_j == F_max - 1 (nsym if none)
        b = nsym;
        while (a < b) {
            const int mid = (a + b) >> 1;
            if ((int)r[mid] - mid >= ftop) b = mid; else a = mid + 1;
        }
        len = a - lo;
        lolen[2 * row] = (uint8_t)lo;
        lolen[2 * row + 1] = (uint8_t)len;
    }
    red[threadIdx.x] = len;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) bsum[blockIdx.x] = red[0];
}

// Exclusive scan of nb block sums in place (one workgroup, chunks of 1024).
__global__ __launch_bounds__(1024) void trim_scan_k(long long* __restrict__ bsum, long long nb) {
    __shared__ long long sh[1024];
    long long carry = 0;
    for (long long base = 0; base < nb; base += 1024) {
        const long long i = base + threadIdx.x;
        const long long v = i < nb ? bsum[i] : 0;
        sh[threadIdx.x] = v;
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {   // inclusive Hillis-Steele scan
            const long long add = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
            __syncthreads();
            sh[threadIdx.x] += add;
            __syncthreads();
        }
        if (i < nb) bsum[i] = carry + sh[threadIdx.x] - v;
        const long long tot = sh[1023];
        __syncthreads();
        carry += tot;
    }
}

__global__ __launch_bounds__(256) void trim_write_k(const uint16_t* __restrict__ cdf, long long n, int nsym,
                                                    const uint8_t* __restrict__ lolen,
                                                    const long long* __restrict__ bsum,
                                                    uint16_t* __restrict__ packed) {
    __shared__ int sh[256];
    const long long row = (long long)blockIdx.x * 256 + threadIdx.x;
    const int len = row < n ? lolen[2 * row + 1] : 0;
    sh[threadIdx.x] = len;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {
        const int add = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
        __syncthreads();
        sh[threadIdx.x] += add;
        __syncthreads();
    }
    if (row < n) {
        const long long off = bsum[blockIdx.x] + sh[threadIdx.x] - len;
        const int lo = lolen[2 * row];
        const uint16_t* r = cdf + row * (nsym + 1);
        for (int t = 0; t < len; ++t) packed[off + t] = (uint16_t)(r[lo + t] - (lo + t));
    }
}

}  // namespace

size_t cdf_trim_scratch_bytes(long long n) { return (size_t)((n + 255) / 256) * sizeof(long long); }

// Block sums of the trim for callers that cannot allocate: one array per GPU, held
// until the process ends.  Host code never passes `trim_scratch` itself (in host code
// the name is not a device address); it passes the address hipGetSymbolAddress gives
// for the current device, looked up once per device.
namespace {
__device__ __align__(256) long long trim_scratch[TRIM_STATIC_SCRATCH_BYTES / sizeof(long long)];
std::mutex g_trim_mu;
long long* g_trim_ptr[TRIM_MAX_DEVICES];
}  // namespace

hipError_t cdf_trim_static_scratch(long long** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= TRIM_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_trim_mu);
    if (!g_trim_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(trim_scratch));
        if (e != hipSuccess) return e;
        g_trim_ptr[dev] = static_cast<long long*>(p);
    }
    *out = g_trim_ptr[dev];
    return hipSuccess;
}

hipError_t launch_cdf_trim(const uint16_t* cdf, long long n, int nsym, uint8_t* lolen, uint16_t* packed,
                           long long* scratch, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const long long nb = (n + 255) / 256;
    hipLaunchKernelGGL(trim_len_k, dim3((unsigned)nb), dim3(256), 0, s, cdf, n, nsym, lolen, scratch);
    hipLaunchKernelGGL(trim_scan_k, dim3(1), dim3(1024), 0, s, scratch, nb);
    hipLaunchKernelGGL(trim_write_k, dim3((unsigned)nb), dim3(256), 0, s, cdf, n, nsym, lolen, scratch, packed);
    return hipGetLastError();
}

}  // namespace wv

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
// What bounds it: vector instructions, about 230 per window entry and 6 per pair of entries filled, and for
// narrow windows the writes (260 bytes a row).  Windows differ: for scales spread over a decade
// their mean is 25 entries, but the longest of 64 rows has 101.  So a workgroup fills its rows' entries
// outside the windows in LDS, deals all the window entries evenly to its threads (a prefix sum of the
// window lengths, a binary search per entry), and copies the rows out as one block.  (One thread or four
// lanes per row step through the longest window of a wave.)  An untrained model's rows all have six
// entries: where a workgroup's windows are of one length, a multiplication takes the search's place.
//   rows (scales)                 a thread or 4 lanes per row   now
//   9.6 M (six entries all)             564 us                  573 us, 5.0 TB/s
//   9.6 M (0.7, spread by 15 %)         706                     646
//   2.4 M (over a decade)              1234                     322
//   1152 (over a decade)                 31                     4.8
// 128 or 512 threads, or 32 rows, were 10 to 20 % slower, four lanes per row with its values in registers
// 8 %.  The running maximum is the identity up to rounding, so entries are only compared with their
// predecessors, and a row is gone through again if one of them is larger.
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
    constexpr bool BIG = ROWS == 64;
    extern __shared__ __attribute__((aligned(16))) uint16_t tab[];   // [ROWS][nsym + 1]
    __shared__ CdfRow<K, DIST> R[ROWS];
    __shared__ int win[ROWS][2];        // evaluated entries j1 <= j < j2
    __shared__ int first[ROWS + 1];     // of a row's entries among the workgroup's
    __shared__ int bad[ROWS], anybad;   // rows whose F decreases somewhere
    __shared__ int common;              // the rows' window length if they have one, else 0
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
        if (BIG) {
            const bool same = __all(len == __builtin_amdgcn_readfirstlane(len));
            if (tid == 0) common = same ? len : 0;
        }
    }
    __syncthreads();
    const int Fmax = 65536 - nsym;
    {   // cdf[j] = j below the window, j + F_max - 1 above it; the last entry 0 (a thread keeps its row)
        const int r = tid % ROWS, q0 = tid / ROWS, j2 = win[r][1];
        if ((E & 1) == 0) {   // two entries at a time; the window's last one, beside the first above it, is replaced below
            uint32_t* w = reinterpret_cast<uint32_t*>(tab) + r * (E / 2);
            const uint32_t above = 0x10001u * (uint32_t)(Fmax - 1);
            uint32_t v = 0x20002u * q0 + 0x10000u;
#pragma unroll 4
            for (int q = q0; q < E / 2; q += NT / ROWS, v += 0x20002u * (NT / ROWS)) w[q] = v + (q >= (j2 >> 1) ? above : 0u);
        } else {
            for (int j = q0; j < nsym; j += NT / ROWS) tab[r * E + j] = (uint16_t)(j + (j >= j2 ? Fmax - 1 : 0));
        }
    }
    __syncthreads();
    if (tid < ROWS) {
        tab[tid * E + nsym] = 0;
        const int j2 = win[tid][1];
        if (win[tid][0] == j2) tab[tid * E + j2 - 1] = (uint16_t)(j2 - 1);   // an empty window: below it
    }
    const int total = first[ROWS], len = BIG ? common : 0;
    const float per = __builtin_amdgcn_rcpf((float)len);
    auto locate = [&](int e, int& r, int& i) {   // entry e is entry i of row r's window
        if (BIG && len) {
            r = (int)(((float)e + 0.5f) * per);   // exact: e < 2^14, so the product is 1/512 or more from a whole number
            i = e - r * len;
            return;
        }
        r = 0;
#pragma unroll
        for (int d = ROWS / 2; d >= 1; d >>= 1)   // last row with first[r] <= e
            if (first[r + d] <= e) r += d;
        i = e - first[r];
    };
    for (int e0 = tid - lane; e0 < total; e0 += NT) {
        int r, i;
        locate(min(e0 + lane, total - 1), r, i);
        const int j = win[r][0] + i;
        const CdfRow<K, DIST> row = R[r];
        const int F = max(cdf_F_in<K, DIST>(row, j), 0);
        tab[r * E + j] = (uint16_t)(j + F);
        // the row's entry before this one, except for the first lane (checked below)
        const int before = __builtin_amdgcn_update_dpp(0, F, 0x138, 0xf, 0xf, false);   // wave_shr:1
        if (lane > 0 && i > 0 && F < before) bad[r] = anybad = 1;
    }
    __syncthreads();
    for (int e = 64 * tid; e < total; e += 64 * NT) {   // entries that a first lane evaluated
        int r, i;
        locate(e, r, i);
        const uint16_t* c = tab + r * E + win[r][0] + i;
        if (i > 0 && c[0] <= c[-1]) bad[r] = anybad = 1;
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
        char* base = reinterpret_cast<char*>(dst);
        const char* from = reinterpret_cast<const char*>(tab);
#pragma unroll 4
        for (uint32_t o = 16 * tid; o < 2u * nel; o += 16 * NT)
            st_g(reinterpret_cast<uint4*>(base + o), *reinterpret_cast<const uint4*>(from + o));
    } else {
        for (int i = tid; i < nel; i += NT) dst[i] = tab[i];
    }
}

}  // namespace

hipError_t launch_cdf(const float* params, long long n, int K, int dist, int smin, int nsym,
                      uint16_t* cdf, hipStream_t s) {
    if (n == 0) return hipSuccess;
    if (nsym + 1 > MAXE || nsym < 2) return hipErrorInvalidValue;
    // 64 rows per workgroup share the fixed work best, but in 16-row workgroups few rows are on more CUs.
    // 16 against 64, scales over a decade: 1152 rows 4.8 and 8.3 us, 18 432 7.5 and 10.4, 49 152 13.4 and
    // 13.7, 98 304 21.5 and 19.8; all windows six entries: 1152 3.7 and 4.3, 18 432 5.1 and 5.3, 49 152 8.9
    // and 6.9, 98 304 14.4 and 9.3.
    const bool small = n <= 40 * 1024;
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

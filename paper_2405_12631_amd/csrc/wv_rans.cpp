// Host rANS entropy coder for the per-coefficient CDF tables.
//
// Byte-wise renormalising range-ANS (J. Duda, 2013): 32-bit state in
// [L, 256 L) with L = 2^23, probabilities out of M = 2^16.  Symbols are
// pushed last to first so that the decoder pops them in raster order; the
// encoder writes bytes downwards from the end of the output buffer and
// finally the state, little endian, in front of them.  A valid stream
// decodes back to the initial state L with every byte consumed, which is
// checked to flag corrupt input.
#include <stdint.h>
#include <string.h>

#include "../../include/wv.h"

namespace {

constexpr uint32_t kL = 1u << 23;
constexpr int kProbBits = 16;
constexpr uint32_t kM = 1u << kProbBits;

inline uint32_t row_at(const uint16_t* row, int s, int nsym) {
    return s >= nsym ? kM : row[s];   // entry nsym is stored as 0 (mod 2^16)
}

// The table of one coder step: its entry s, and the symbol of a slot (the largest s with
// at(s) <= slot; at(0) = 0, at(nsym) = M).
template <class Entry>
int bisect(const Entry& entry, int nsym, uint32_t slot) {
    int lo = 0, hi = nsym;   // invariant: entry(lo) <= slot < entry(hi), with entry(nsym) = M never read
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (entry(mid) <= slot)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}
struct FullRow {
    const uint16_t* row;
    int nsym;
    uint32_t at(int s) const { return row_at(row, s, nsym); }
    int find(uint32_t slot) const {
        return bisect([this](int s) { return row[s]; }, nsym, slot);
    }
};
// A trimmed row used as it is: outside the window an entry and a symbol are known from (lo, len)
// alone, so a symbol costs a search over the window (about ten values, halved without branches)
// instead of the 129 entries of a rebuilt row (73 -> 20 ns a symbol with the model of 512 x 768).
struct TrimRow {
    const uint16_t* f;   // F_lo .. F_{lo + len - 1}
    int lo, len, nsym, ftop;
    uint32_t at(int s) const {
        if (s >= nsym) return kM;
        return (uint16_t)(s + (s < lo ? 0 : s < lo + len ? f[s - lo] : ftop));
    }
    int find(uint32_t slot) const {
        if (slot < at(lo)) return (int)slot < lo ? (int)slot : lo - 1;
        const int above = lo + len;
        if (slot >= at(above)) {   // above < nsym, since at(nsym) = M
            const int s = (int)slot - ftop;
            return s < nsym ? s : nsym - 1;
        }
        int k = 0;   // last k with lo + k + f[k] <= slot; f[0] qualifies
        for (int n = len; n > 1;) {
            const int half = n >> 1;
            k += (uint16_t)(lo + k + half + f[k + half]) <= slot ? half : 0;
            n -= half;
        }
        return lo + k;
    }
};
// The same row searched as a full one.  In a row whose F falls somewhere (no wv_cdf_trim makes one) a slot
// may lie in several symbols, and the two searches find different ones.
struct TrimRowBisected : TrimRow {
    int find(uint32_t slot) const {
        return bisect([this](int s) { return at(s); }, nsym, slot);
    }
};

// Trimmed tables (wv_cdf_trim): row i as (lo, len) and its F values (build: written out in full),
// which start at offset off of packed; false if they do not describe a row.
struct TrimRows {
    const uint8_t* lolen;
    const uint16_t* packed;
    long long count;   // values in packed
    int nsym;
    bool row(long long i, long long off, TrimRow& r) const {
        const int lo = lolen[2 * i], len = lolen[2 * i + 1];
        if (lo < 1 || lo + len > nsym || off < 0 || off + len > count) return false;
        r.f = packed + off;
        r.lo = lo;
        r.len = len;
        r.nsym = nsym;
        r.ftop = (int)kM - nsym - 1;   // F_max - 1: the plateau above the window
        return true;
    }
    bool build(long long i, long long off, uint16_t* tmp) const {
        const int lo = lolen[2 * i], len = lolen[2 * i + 1];
        if (lo < 1 || lo + len > nsym || off < 0 || off + len > count) return false;
        const int ftop = (int)kM - nsym - 1;   // F_max - 1: the plateau above the window
        for (int j = 0; j < nsym; ++j) {
            const int F = j < lo ? 0 : j < lo + len ? packed[off + j - lo] : ftop;
            tmp[j] = (uint16_t)(j + F);
        }
        return true;
    }
};

}  // namespace

extern "C" int wv_cdf_untrim(const uint8_t* lolen, const uint16_t* packed, long long packed_count, int nsym,
                             long long n, uint16_t* cdf_out) {
    if (nsym < 2 || nsym > 255 || n < 0 || packed_count < 0 || (n > 0 && (!lolen || !cdf_out)) ||
        (packed_count > 0 && !packed))
        return WV_EINVAL;
    TrimRows T{lolen, packed, packed_count, nsym};
    long long off = 0;
    for (long long i = 0; i < n; ++i) {
        uint16_t* row = cdf_out + (size_t)i * (nsym + 1);
        if (!T.build(i, off, row)) return WV_ECORRUPT;
        row[nsym] = 0;   // 2^16 mod 2^16
        off += lolen[2 * i + 1];
    }
    return off == packed_count ? WV_OK : WV_ECORRUPT;
}

namespace {

// Symbols i = n-1 .. 0; row(i, r) sets r to row i's table, false if there is none.
template <class Row, class RowOf>
int encode_rows(RowOf&& rowof, int nsym, const uint8_t* sym, long long n, uint8_t* out, size_t cap, size_t* len) {
    uint8_t* ptr = out + cap;
    uint32_t x = kL;
    for (long long i = n - 1; i >= 0; --i) {
        Row row;
        if (!rowof(i, row)) return WV_EINVAL;
        const int s = sym[i];
        if (s >= nsym) return WV_EINVAL;
        const uint32_t start = row.at(s);
        const uint32_t end = row.at(s + 1);
        if (end <= start) return WV_EINVAL;   // zero-frequency symbol: not encodable
        const uint32_t freq = end - start;
        const uint32_t x_max = ((kL >> kProbBits) << 8) * freq;
        while (x >= x_max) {
            if (ptr == out) return WV_ENOMEM;
            *--ptr = (uint8_t)(x & 0xff);
            x >>= 8;
        }
        x = ((x / freq) << kProbBits) + (x % freq) + start;
    }
    if ((size_t)(ptr - out) < 4) return WV_ENOMEM;
    ptr -= 4;
    ptr[0] = (uint8_t)(x);
    ptr[1] = (uint8_t)(x >> 8);
    ptr[2] = (uint8_t)(x >> 16);
    ptr[3] = (uint8_t)(x >> 24);
    const size_t total = (size_t)(out + cap - ptr);
    memmove(out, ptr, total);
    *len = total;
    return WV_OK;
}

// Symbols i = 0 .. n-1; row(i, r) as above.
template <class Row, class RowOf>
int decode_rows(RowOf&& rowof, long long n, const uint8_t* in, size_t len, uint8_t* sym_out) {
    if (len < 4) return WV_ECORRUPT;
    uint32_t x = (uint32_t)in[0] | ((uint32_t)in[1] << 8) | ((uint32_t)in[2] << 16) | ((uint32_t)in[3] << 24);
    size_t pos = 4;
    if (x < kL) return WV_ECORRUPT;
    for (long long i = 0; i < n; ++i) {
        Row row;
        if (!rowof(i, row)) return WV_ECORRUPT;
        const uint32_t slot = x & (kM - 1);
        const int lo = row.find(slot);
        const uint32_t start = row.at(lo);
        const uint32_t end = row.at(lo + 1);
        if (end <= start || slot < start) return WV_ECORRUPT;
        x = (end - start) * (x >> kProbBits) + slot - start;
        while (x < kL) {
            if (pos >= len) return WV_ECORRUPT;
            x = (x << 8) | in[pos++];
        }
        sym_out[i] = (uint8_t)lo;
    }
    if (x != kL || pos != len) return WV_ECORRUPT;
    return WV_OK;
}

}  // namespace

extern "C" int wv_rans_encode(const uint16_t* cdf, int nsym, const uint8_t* sym, long long n,
                              uint8_t* out, size_t cap, size_t* len) {
    if (nsym < 2 || nsym > 255 || n < 0 || !len || (n > 0 && (!cdf || !sym)) || !out)
        return WV_EINVAL;
    return encode_rows<FullRow>(
        [&](long long i, FullRow& r) {
            r = FullRow{cdf + (size_t)i * (nsym + 1), nsym};
            return true;
        },
        nsym, sym, n, out, cap, len);
}

extern "C" int wv_rans_decode(const uint16_t* cdf, int nsym, long long n, const uint8_t* in,
                              size_t len, uint8_t* sym_out) {
    if (nsym < 2 || nsym > 255 || n < 0 || (n > 0 && (!cdf || !sym_out)) || (len > 0 && !in))
        return WV_EINVAL;
    return decode_rows<FullRow>(
        [&](long long i, FullRow& r) {
            r = FullRow{cdf + (size_t)i * (nsym + 1), nsym};
            return true;
        },
        n, in, len, sym_out);
}

extern "C" int wv_rans_encode_trim(const uint8_t* lolen, const uint16_t* packed, long long packed_count, int nsym,
                                   const uint8_t* sym, long long n, uint8_t* out, size_t cap, size_t* len) {
    if (nsym < 2 || nsym > 255 || n < 0 || packed_count < 0 || !len || (n > 0 && (!lolen || !sym)) || !out ||
        (packed_count > 0 && !packed))
        return WV_EINVAL;
    long long total = 0;
    for (long long i = 0; i < n; ++i) total += lolen[2 * i + 1];
    if (total != packed_count) return WV_EINVAL;
    const TrimRows T{lolen, packed, packed_count, nsym};
    long long end = total;   // rows are visited last to first
    return encode_rows<TrimRow>(
        [&](long long i, TrimRow& r) {
            end -= lolen[2 * i + 1];
            return T.row(i, end, r);
        },
        nsym, sym, n, out, cap, len);
}

extern "C" int wv_rans_decode_trim(const uint8_t* lolen, const uint16_t* packed, long long packed_count, int nsym,
                                   long long n, const uint8_t* in, size_t len, uint8_t* sym_out) {
    if (nsym < 2 || nsym > 255 || n < 0 || packed_count < 0 || (n > 0 && (!lolen || !sym_out)) ||
        (len > 0 && !in) || (packed_count > 0 && !packed))
        return WV_EINVAL;
    const TrimRows T{lolen, packed, packed_count, nsym};
    auto decode = [&](auto kind) {
        using Row = decltype(kind);
        long long off = 0;   // rows are visited first to last
        return decode_rows<Row>(
            [&](long long i, Row& r) {
                const bool ok = T.row(i, off, r);
                off += lolen[2 * i + 1];
                return ok;
            },
            n, in, len, sym_out);
    };
    // A stream that fails is decoded again as the full tables would decode it, so that none is refused
    // that wv_rans_decode takes.
    const int rc = decode(TrimRow{});
    return rc == WV_ECORRUPT ? decode(TrimRowBisected{}) : rc;
}

// Host-side construction of the dictionary form of a CRS matrix (the
// CsrView::code and CsrView::ccode arrays): distinct column offsets,
// distinct values, codes and value tables.  Used for the solver matrices of
// a handle and for the operators of an AMG hierarchy's levels.
#pragma once

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <numeric>
#include <thread>
#include <vector>

#include "core.h"

namespace mrhs {
namespace dict {

// Distinct keys in order of first appearance, at most `limit`; open
// addressing over a power-of-two table.
template <typename K>
struct KeySet {
    std::vector<K> keys;
    std::vector<int32_t> slot;  // index into keys + 1, 0 empty
    uint64_t mask = 0;
    explicit KeySet(int limit)
    {
        size_t cap = 16;
        while (cap < 4 * static_cast<size_t>(limit))
            cap *= 2;
        slot.assign(cap, 0);
        mask = cap - 1;
    }
    // MurmurHash3's 64-bit finalizer: every key bit reaches the low bits the
    // table uses (values such as 4 + k 2^-10 have zero low mantissa bits)
    static uint64_t hash(K k)
    {
        uint64_t z = static_cast<uint64_t>(k);
        z ^= z >> 33;
        z *= 0xff51afd7ed558ccdull;
        z ^= z >> 33;
        z *= 0xc4ceb9fe1a85ec53ull;
        return z ^ (z >> 33);
    }
    // index of k, inserting it; -1 when that would exceed limit
    int32_t add(K k, int limit)
    {
        for (uint64_t h = hash(k) & mask;; h = (h + 1) & mask) {
            const int32_t e = slot[h];
            if (!e) {
                if (static_cast<int>(keys.size()) >= limit)
                    return -1;
                keys.push_back(k);
                slot[h] = static_cast<int32_t>(keys.size());
                return slot[h] - 1;
            }
            if (keys[e - 1] == k)
                return e - 1;
        }
    }
    int32_t find(K k) const
    {
        for (uint64_t h = hash(k) & mask;; h = (h + 1) & mask) {
            const int32_t e = slot[h];
            if (!e || keys[e - 1] == k)
                return e - 1;
        }
    }
};

inline int threads()
{
    const unsigned hw = std::thread::hardware_concurrency();
    return std::max(1, std::min(16, static_cast<int>(hw ? hw : 1)));
}

// Runs fn(lo, hi, t) over T contiguous row ranges of [0, n) in threads.
template <class F>
void row_ranges(int32_t n, int T, F &&fn)
{
    std::vector<std::thread> th;
    for (int t = 0; t < T; ++t) {
        const int32_t lo = static_cast<int32_t>(static_cast<int64_t>(n) * t / T);
        const int32_t hi = static_cast<int32_t>(static_cast<int64_t>(n) * (t + 1) / T);
        th.emplace_back([&fn, lo, hi, t] { fn(lo, hi, t); });
    }
    for (auto &x : th)
        x.join();
}

// Distinct keys of key(i, j) over the entries j of rows i in [0, n), in order
// of first appearance in row order, at most limit (false when there are more).
template <typename K, class KeyOf>
bool distinct_keys(int32_t n, const int32_t *rp, int limit, KeyOf key, KeySet<K> &out)
{
    const int T = threads();
    std::vector<KeySet<K>> local(T, KeySet<K>(limit));
    std::vector<char> over(T, 0);
    row_ranges(n, T, [&](int32_t lo, int32_t hi, int t) {
        for (int32_t i = lo; i < hi && !over[t]; ++i)
            for (int32_t j = rp[i]; j < rp[i + 1]; ++j)
                if (local[t].add(key(i, j), limit) < 0) {
                    over[t] = 1;
                    break;
                }
    });
    for (int t = 0; t < T; ++t) {
        if (over[t])
            return false;
        for (K k : local[t].keys)
            if (out.add(k, limit) < 0)
                return false;
    }
    return true;
}

template <typename V>
struct BitsOf;
template <>
struct BitsOf<double> {
    using U = uint64_t;
};
template <>
struct BitsOf<float> {
    using U = uint32_t;
};

// The distinct column offsets col - row of a matrix when there are at most
// kDictOffs of them (ok), with the bits ob of an offset index.
struct Offsets {
    KeySet<int64_t> set{kDictOffs};
    bool ok = false;
    int ob = 0;
};

inline void offsets(int32_t n, const int32_t *rp, const int32_t *ci, Offsets &o)
{
    auto off = [&](int32_t i, int32_t j) { return static_cast<int64_t>(ci[j]) - i; };
    o.ok = distinct_keys<int64_t>(n, rp, kDictOffs, off, o.set);
    o.ob = 0;
    while (o.ok && (1 << o.ob) < static_cast<int>(o.set.keys.size()))
        ++o.ob;
}

// Codes of one value array hv over the entries of a matrix: 16-bit codes
// (value index << ob | offset index, 8 codes of padding) when the offsets
// fit, else 32-bit column codes (value index << cb | column, 4 codes of
// padding) when the columns fit beside the value index; ok = false when the
// array has more than kDictVals distinct values (bit patterns) or neither
// form applies.
template <typename V>
struct Codes {
    bool ok = false;
    std::vector<uint16_t> code;
    std::vector<uint32_t> ccode;
    std::vector<V> tab;
    int cb = 0;
};

template <typename V>
Codes<V> codes(int32_t n, int64_t nnz, const int32_t *rp, const int32_t *ci, const V *hv, const Offsets &offs)
{
    using U = typename BitsOf<V>::U;
    Codes<V> out;
    const int limit = offs.ok ? std::min(kDictVals, 1 << (16 - offs.ob)) : kDictVals;
    KeySet<U> vals(limit);
    auto bits = [&](int32_t, int32_t j) {
        U u;
        std::memcpy(&u, &hv[j], sizeof(U));
        return u;
    };
    if (!distinct_keys<U>(n, rp, limit, bits, vals))
        return out;
    if (!offs.ok) {
        int vb = 1;  // at least one bit, so the column field is at most 31 bits
        while ((1 << vb) < static_cast<int>(vals.keys.size()))
            ++vb;
        out.cb = 32 - vb;
        if (static_cast<int64_t>(n) > (static_cast<int64_t>(1) << out.cb))
            return out;
    }
    const size_t ncode = static_cast<size_t>(nnz) + (offs.ok ? 8 : 4);
    if (offs.ok)
        out.code.assign(ncode, 0);
    else
        out.ccode.assign(ncode, 0);
    row_ranges(n, threads(), [&](int32_t lo, int32_t hi, int) {
        for (int32_t i = lo; i < hi; ++i)
            for (int32_t j = rp[i]; j < rp[i + 1]; ++j) {
                const uint32_t v = static_cast<uint32_t>(vals.find(bits(i, j)));
                if (offs.ok)
                    out.code[j] = static_cast<uint16_t>((v << offs.ob) |
                                                        offs.set.find(static_cast<int64_t>(ci[j]) - i));
                else
                    out.ccode[j] = (v << out.cb) | static_cast<uint32_t>(ci[j]);
            }
    });
    out.tab.resize(vals.keys.size());
    std::memcpy(out.tab.data(), vals.keys.data(), sizeof(V) * out.tab.size());
    out.ok = true;
    return out;
}

// The row-pattern form (CsrView::pid) of a matrix whose two value arrays
// both have 16-bit codes c0 and c1: rows with equal code sequences share a
// pattern, numbered by first appearance.  ok = false when there are more
// than kPatMax patterns, more than one pattern per kPatRowsPer rows (the
// table would rival the codes it replaces: 16 bytes per entry of a pattern
// against 2 per entry of every row), or a table past kPatEntries entries.
struct Patterns {
    bool ok = false;
    int32_t pk = 0;               // entries per pattern in the table (whole batches)
    int32_t run = 0;              // mean run of rows with one pattern
    std::vector<uint16_t> id;     // [n]
    std::vector<int32_t> rep;     // a row of each pattern
    std::vector<int32_t> len;     // its entries
};

// Distinct rows of a range, in order of first appearance.
class RowSet {
  public:
    RowSet(const int32_t *rp, const uint16_t *c0, const uint16_t *c1) : rp_(rp), c0_(c0), c1_(c1)
    {
        slot_.assign(4 * kPatMax, 0);
    }
    std::vector<int32_t> rows;
    bool same(int32_t a, int32_t b) const
    {
        const size_t na = rp_[a + 1] - rp_[a], nb = rp_[b + 1] - rp_[b];
        return na == nb && std::memcmp(c0_ + rp_[a], c0_ + rp_[b], 2 * na) == 0 &&
               std::memcmp(c1_ + rp_[a], c1_ + rp_[b], 2 * na) == 0;
    }
    // index of row i's pattern, inserting it; -1 when that would be the
    // (kPatMax + 1)-th
    int32_t add(int32_t i)
    {
        uint64_t h = static_cast<uint64_t>(rp_[i + 1] - rp_[i]);
        for (int32_t j = rp_[i]; j < rp_[i + 1]; ++j)
            h = KeySet<uint64_t>::hash(h ^ (static_cast<uint64_t>(c0_[j]) << 32 | c1_[j]));
        for (uint64_t k = h & (slot_.size() - 1);; k = (k + 1) & (slot_.size() - 1)) {
            if (!slot_[k]) {
                if (rows.size() >= static_cast<size_t>(kPatMax))
                    return -1;
                rows.push_back(i);
                slot_[k] = static_cast<int32_t>(rows.size());
                return slot_[k] - 1;
            }
            if (same(rows[slot_[k] - 1], i))
                return slot_[k] - 1;
        }
    }

  private:
    const int32_t *rp_;
    const uint16_t *c0_, *c1_;
    std::vector<int32_t> slot_;
};

inline Patterns patterns(int32_t n, const int32_t *rp, const uint16_t *c0, const uint16_t *c1)
{
    Patterns out;
    const int T = threads();
    std::vector<RowSet> local(T, RowSet(rp, c0, c1));
    std::vector<char> over(T, 0);
    out.id.resize(static_cast<size_t>(n));
    row_ranges(n, T, [&](int32_t lo, int32_t hi, int t) {
        for (int32_t i = lo; i < hi; ++i) {  // most rows repeat the one before
            if (i > lo && local[t].same(i - 1, i)) {
                out.id[i] = out.id[i - 1];
                continue;
            }
            const int32_t k = local[t].add(i);
            if (k < 0) {
                over[t] = 1;
                return;
            }
            out.id[i] = static_cast<uint16_t>(k);
        }
    });
    RowSet all(rp, c0, c1);
    std::vector<std::vector<uint16_t>> map(T);
    for (int t = 0; t < T; ++t) {
        if (over[t])
            return out;
        for (int32_t r : local[t].rows) {
            const int32_t k = all.add(r);
            if (k < 0)
                return out;
            map[t].push_back(static_cast<uint16_t>(k));
        }
    }
    int32_t longest = 0;
    for (int32_t r : all.rows) {
        out.len.push_back(rp[r + 1] - rp[r]);
        longest = std::max(longest, out.len.back());
    }
    auto whole = [&](int32_t nb) { return std::max(1, (longest + nb - 1) / nb) * nb; };
    out.pk = std::max(whole(kPatBatch), whole(MRHS_GATHER_BATCH));
    const int64_t npat = static_cast<int64_t>(all.rows.size());
    if (npat * kPatRowsPer > n || npat * out.pk > kPatEntries)
        return out;
    std::vector<int32_t> runs(T, 0);
    row_ranges(n, T, [&](int32_t lo, int32_t hi, int t) {
        int32_t count = 0;
        for (int32_t i = lo; i < hi; ++i) {
            out.id[i] = map[t][out.id[i]];
            count += i == lo || out.id[i] != out.id[i - 1];
        }
        runs[t] = count;
    });
    out.run = static_cast<int32_t>(n / std::max<int64_t>(1, std::accumulate(runs.begin(), runs.end(), int64_t{0})));
    out.rep = all.rows;
    out.ok = true;
    return out;
}

// The table of one value array: each pattern's entries from its
// representative row, padded with entries of the row itself and value 0.
inline std::vector<PatEntry<double>> pattern_table(const Patterns &p, const int32_t *rp, const int32_t *ci,
                                                   const double *hv)
{
    std::vector<PatEntry<double>> tab(p.rep.size() * static_cast<size_t>(p.pk), PatEntry<double>{0.0, 0, 0});
    for (size_t k = 0; k < p.rep.size(); ++k)
        for (int32_t j = 0; j < p.len[k]; ++j) {
            PatEntry<double> &e = tab[k * p.pk + j];
            e.v = hv[rp[p.rep[k]] + j];
            e.off = ci[rp[p.rep[k]] + j] - p.rep[k];
        }
    return tab;
}

inline std::vector<PatEntry<float>> round_table(const std::vector<PatEntry<double>> &tab)
{
    std::vector<PatEntry<float>> out;
    out.reserve(tab.size());
    for (const PatEntry<double> &e : tab)
        out.push_back(PatEntry<float>{static_cast<float>(e.v), e.off});
    return out;
}

// The patterns of stencil shape (PatStencil): at most kFar distant entries,
// the near ones (offsets -1, 0, 1, each at most once and in this order)
// together among them.
template <typename V>
std::vector<PatStencil<V>> stencil_table(const Patterns &p, const std::vector<PatEntry<V>> &tab)
{
    std::vector<PatStencil<V>> out(p.rep.size());
    std::memset(static_cast<void *>(out.data()), 0, sizeof(PatStencil<V>) * out.size());
    for (size_t k = 0; k < p.rep.size(); ++k) {
        PatStencil<V> s{};
        int far = 0, before = -1, last = -2;
        bool has[3] = {false, false, false}, ok = true, left = false;  // left: past the near entries
        for (int32_t j = 0; j < p.len[k] && ok; ++j) {
            const PatEntry<V> &e = tab[k * p.pk + j];
            if (e.off >= -1 && e.off <= 1) {
                ok = !left && e.off > last;
                last = e.off;
                if (before < 0)
                    before = far;
                has[e.off + 1] = true;
                s.nv[e.off + 1] = e.v;
            } else {
                left = before >= 0;
                ok = far < kFar;
                if (ok) {
                    s.fo[far] = e.off;
                    s.fv[far] = e.v;
                    ++far;
                }
            }
        }
        if (!ok)
            continue;
        s.meta = PatStencil<V>::pack(before < 0 ? far : before, far, has[0], has[1], has[2]);
        out[k] = s;
    }
    return out;
}

} // namespace dict
} // namespace mrhs

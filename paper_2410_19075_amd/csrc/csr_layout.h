// Host layout of a CSR network's in-edges for the gather kernel (csr.hip).
#pragma once

#include <algorithm>
#include <cstdint>
#include <memory>
#include <vector>

#include "nd_dev.h"

namespace nd {

template <class KT>
struct CsrLayout {
    std::vector<int64_t> bptr;        // per source block b, row offsets at [b*(n+1), (b+1)*(n+1))
    std::unique_ptr<uint32_t[]> col;  // edges, block-major (csr_packed)
    std::unique_ptr<KT[]> w;          // their weights
    int edges = 1;                    // edges of the largest chunk
};

// Sorts up to kCsrChunk edges by source, stably: one counting pass over the bits of a
// block's sources, two over half of them where one would have more buckets than the
// fullest chunk has edges (and than 512).
class CsrChunkSort {
public:
    CsrChunkSort(int64_t n, int edges) : a_(edges), t_(edges) {
        int bits = 1;
        while (((n + kCsrSourceBlocks - 1) / kCsrSourceBlocks - 1) >> bits) ++bits;
        passes_ = (1 << bits) > std::max(512, edges) ? 2 : 1;
        bits_ = (bits + passes_ - 1) / passes_;
        for (auto& c : cnt_) c.resize(size_t(1) << bits_);
    }
    // src: m <= edges sources relative to the block's first; returns the edges, source << kCsrSlotBits |
    // place in src, by ascending source
    const uint32_t* operator()(const uint32_t* src, int m) {
        const uint32_t mask = (1u << bits_) - 1;
        for (int k = 0; k < passes_; ++k) std::fill(cnt_[k].begin(), cnt_[k].end(), 0);
        if (passes_ == 1) {
            for (int q = 0; q < m; ++q) ++cnt_[0][src[q]];
            offsets(cnt_[0]);
            for (int q = 0; q < m; ++q) a_[cnt_[0][src[q]]++] = src[q] << kCsrSlotBits | (uint32_t)q;
            return a_.data();
        }
        for (int q = 0; q < m; ++q) {
            ++cnt_[0][src[q] & mask];
            ++cnt_[1][src[q] >> bits_];
        }
        for (auto& c : cnt_) offsets(c);
        for (int q = 0; q < m; ++q) t_[cnt_[0][src[q] & mask]++] = src[q] << kCsrSlotBits | (uint32_t)q;
        for (int q = 0; q < m; ++q) a_[cnt_[1][t_[q] >> (kCsrSlotBits + bits_)]++] = t_[q];
        return a_.data();
    }

private:
    static void offsets(std::vector<int>& c) {
        int o = 0;
        for (int& v : c) {
            const int k = v;
            v = o;
            o += k;
        }
    }
    int bits_, passes_;
    std::vector<uint32_t> a_, t_;
    std::vector<int> cnt_[2];
};

// Entries of c[0 .. m) that are at least v.
inline int64_t count_from(const int32_t* c, int64_t m, int32_t v) {
    int64_t k = 0;
    for (int64_t e0 = 0; e0 < m; e0 += 1 << 20) {
        int32_t s = 0;
        const int64_t e1 = std::min<int64_t>(m, e0 + (1 << 20));
        for (int64_t e = e0; e < e1; ++e) s += c[e] >= v;
        k += s;
    }
    return k;
}

inline bool ascending(const int32_t* c, int64_t m) {
    int32_t down = 0;
    for (int64_t e = 1; e < m; ++e) down |= c[e] < c[e - 1];
    return !down;
}

// Split every row's in-edges by source block, each block's in the row's order, lay the
// blocks out one after the other, and sort the edges of every chunk by source
// (networks whose edges pack).  A tile's edges are split into buffers that stay in
// cache and leave them once, sorted, so the edge arrays are written in one pass.
// Bound: the reads of the rows and the page faults of the fresh edge arrays.  nd_create
// of 2e5 neurons of degree 100 / of degree 10 / of 2000 neurons of degree 10: 121 / 22 /
// 0.25 ms; with the arrays filled in row order and sorted afterwards in two passes of
// 1024 buckets 174 / 38 / 0.37 ms, filled and not sorted 151 / 21 / 0.21 ms.
template <class KT>
CsrLayout<KT> csr_layout(int64_t n, const int64_t* row_ptr, const int32_t* col, const double* weight) {
    constexpr int B = kCsrSourceBlocks;
    const int64_t nnz = row_ptr[n], rows = csr_rows(n);
    const bool packed = csr_packed(n);
    CsrLayout<KT> L;
    L.bptr.assign((size_t)B * (n + 1), 0);
    L.col.reset(new uint32_t[std::max<int64_t>(nnz, 1)]);  // (not cleared: written below)
    L.w.reset(new KT[std::max<int64_t>(nnz, 1)]);
    int32_t begin[B + 1];  // first source of each block
    for (int b = 0; b <= B; ++b) begin[b] = (int32_t)csr_block_begin(b, n);
    // edges of each block by row: differences of the counts of sources from a block's
    // begin on (passes over a row without branches)
    for (int64_t i = 0; i < n; ++i) {
        const int32_t* c = col + row_ptr[i];
        const int64_t m = row_ptr[i + 1] - row_ptr[i];
        int64_t from = m;
        for (int b = 0; b < B; ++b) {
            int64_t next = 0;
            if (b + 1 < B) next = count_from(c, m, begin[b + 1]);
            L.bptr[(size_t)b * (n + 1) + i + 1] = from - next;
            from = next;
        }
    }
    int64_t base = 0, widest = 0;  // edges of the fullest (row tile, block)
    for (int b = 0; b < B; ++b) {
        int64_t* p = L.bptr.data() + (size_t)b * (n + 1);
        p[0] = base;
        for (int64_t i = 0; i < n; ++i) p[i + 1] += p[i];
        base = p[n];
        for (int64_t r0 = 0; r0 < n; r0 += rows) widest = std::max(widest, p[std::min(r0 + rows, n)] - p[r0]);
    }
    L.edges = (int)std::min<int64_t>(kCsrChunk, std::max<int64_t>(1, widest));
    CsrChunkSort sort(n, L.edges);
    int64_t fullest = 0;  // edges of the fullest row tile
    for (int64_t r0 = 0; r0 < n; r0 += rows) fullest = std::max(fullest, row_ptr[std::min(r0 + rows, n)] - row_ptr[r0]);
    std::vector<uint32_t> tc(fullest);
    std::vector<KT> tw(fullest);
    for (int64_t r0 = 0; r0 < n; r0 += rows) {
        const int64_t r1 = std::min(r0 + rows, n);
        uint32_t* pc[B];
        KT* pw[B];
        for (int64_t b = 0, o = 0; b < B; ++b) {
            pc[b] = tc.data() + o;
            pw[b] = tw.data() + o;
            o += L.bptr[(size_t)b * (n + 1) + r1] - L.bptr[(size_t)b * (n + 1) + r0];
        }
        for (int64_t i = r0; i < r1; ++i) {
            const int32_t* c = col + row_ptr[i];
            const double* wt = weight + row_ptr[i];
            const int64_t m = row_ptr[i + 1] - row_ptr[i];
            if (ascending(c, m)) {  // (usual) a block's edges are consecutive
                for (int b = 0; b < B; ++b) {
                    const int64_t* p = L.bptr.data() + (size_t)b * (n + 1) + i;
                    const int64_t k = p[1] - p[0];
                    const int32_t first = packed ? begin[b] : 0;
                    for (int64_t q = 0; q < k; ++q) {
                        pc[b][q] = (uint32_t)(c[q] - first);
                        pw[b][q] = (KT)wt[q];
                    }
                    pc[b] += k;
                    pw[b] += k;
                    c += k;
                    wt += k;
                }
            } else {
                for (int64_t q = 0; q < m; ++q) {
                    int b = 0;
                    while (c[q] >= begin[b + 1]) ++b;
                    *pc[b]++ = (uint32_t)(c[q] - (packed ? begin[b] : 0));
                    *pw[b]++ = (KT)wt[q];
                }
            }
        }
        for (int b = 0; b < B; ++b) {
            const int64_t* p = L.bptr.data() + (size_t)b * (n + 1);
            const int64_t m = p[r1] - p[r0];
            const uint32_t* sc = pc[b] - m;  // (advanced to the end above)
            const KT* sw = pw[b] - m;
            uint32_t* dc = L.col.get() + p[r0];
            KT* dw = L.w.get() + p[r0];
            if (!packed) {
                std::copy(sc, sc + m, dc);
                std::copy(sw, sw + m, dw);
                continue;
            }
            for (int64_t c0 = 0; c0 < m; c0 += kCsrChunk) {
                const int k = (int)std::min<int64_t>(kCsrChunk, m - c0);
                const uint32_t* a = sort(sc + c0, k);
                for (int q = 0; q < k; ++q) {
                    dc[c0 + q] = a[q];
                    dw[c0 + q] = sw[c0 + (a[q] & (kCsrChunk - 1))];
                }
            }
        }
    }
    return L;
}

}  // namespace nd

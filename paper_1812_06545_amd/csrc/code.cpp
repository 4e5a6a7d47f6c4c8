// Code handles: validation of H and its device-resident layouts.
//
// H (arxiv 1812.06545, Section II) arrives as CSR or as a quasi-cyclic base
// matrix of circulant shifts.  Both are canonicalised to CSR with columns
// ascending inside each row, and the transposed view (each column's edges in
// ascending row order) is built once; everything is uploaded in a single
// device allocation and never changes afterwards.
#include <algorithm>
#include <cstring>
#include <vector>

#include "ldpc_internal.h"

namespace {

struct HostLayout {
    int32_t m = 0, n = 0;
    std::vector<int32_t> row_ptr, col_idx, col_ptr, col_edge;
    int32_t max_row_deg = 0, max_col_deg = 0;
};

ldpc_status build_host_layout(int32_t m, int32_t n, const int32_t *row_ptr, const int32_t *col_idx,
                              HostLayout &h)
{
    if (m < 1 || n < 1 || !row_ptr)
        return LDPC_EINVAL;
    if (row_ptr[0] != 0)
        return LDPC_EINVAL;
    for (int32_t i = 0; i < m; ++i)
        if (row_ptr[i + 1] < row_ptr[i])
            return LDPC_EINVAL;
    const int64_t E = row_ptr[m];
    if (E > 0 && !col_idx)
        return LDPC_EINVAL;
    // The kernels index a 64-frame chunk's messages and posteriors with
    // 32-bit byte and element offsets (edge x 64, variable x 64 x 8 bytes).
    if (E > LDPC_MAX_EDGES || n > LDPC_MAX_VARIABLES)
        return LDPC_EUNSUPPORTED;
    h.m = m;
    h.n = n;
    h.row_ptr.assign(row_ptr, row_ptr + m + 1);
    h.col_idx.assign(col_idx, col_idx + E);
    for (int32_t i = 0; i < m; ++i) {
        const int32_t b = row_ptr[i], e = row_ptr[i + 1];
        int32_t last = -1;
        bool ascending = true;
        for (int32_t k = b; k < e; ++k) {
            const int32_t c = col_idx[k];
            if (c < 0 || c >= n)
                return LDPC_EINVAL;
            ascending &= c > last;
            last = c;
        }
        if (!ascending) {
            std::sort(h.col_idx.begin() + b, h.col_idx.begin() + e);
            for (int32_t k = b + 1; k < e; ++k)
                if (h.col_idx[k] == h.col_idx[k - 1])
                    return LDPC_EINVAL;  // duplicate edge
        }
        h.max_row_deg = std::max(h.max_row_deg, e - b);
    }
    if (h.max_row_deg > LDPC_MAX_ROW_DEGREE)
        return LDPC_EUNSUPPORTED;
    h.col_ptr.assign(n + 1, 0);
    for (int64_t k = 0; k < E; ++k)
        h.col_ptr[h.col_idx[k] + 1]++;
    for (int32_t j = 0; j < n; ++j) {
        h.max_col_deg = std::max(h.max_col_deg, h.col_ptr[j + 1]);
        h.col_ptr[j + 1] += h.col_ptr[j];
    }
    h.col_edge.resize(E);
    std::vector<int32_t> next(h.col_ptr.begin(), h.col_ptr.end() - 1);
    for (int32_t k = 0; k < static_cast<int32_t>(E); ++k)  // E is at most LDPC_MAX_EDGES
        h.col_edge[next[h.col_idx[k]]++] = k;
    return LDPC_OK;
}

// Greedy layers over the rows in ascending order: a row opens a new layer
// when it shares a variable with a row of the current one.  Visiting the
// layers in order, each as a parallel step, equals visiting the rows one at a
// time in order.
void layer_tables(const HostLayout &h, std::vector<int32_t> &layer_ptr, std::vector<int32_t> &layer_dmax)
{
    std::vector<int32_t> mark(h.n, -1);
    int32_t cur = 0;
    layer_ptr.assign(1, 0);
    layer_dmax.assign(1, 0);
    for (int32_t i = 0; i < h.m; ++i) {
        const int32_t b = h.row_ptr[i], e = h.row_ptr[i + 1];
        bool clash = false;
        for (int32_t k = b; k < e && !clash; ++k)
            clash = mark[h.col_idx[k]] == cur;
        if (clash) {
            ++cur;
            layer_ptr.push_back(i);
            layer_dmax.push_back(0);
        }
        for (int32_t k = b; k < e; ++k)
            mark[h.col_idx[k]] = cur;
        layer_dmax.back() = std::max(layer_dmax.back(), e - b);
    }
    layer_ptr.push_back(h.m);
    if (h.m == 0) {
        layer_ptr.assign(1, 0);
        layer_dmax.clear();
    }
}

// FNV-1a over the code's sizes, lifting size and row and column degree
// histograms: codes of one shape (whatever their edge placement) share it.
uint64_t shape_hash(const HostLayout &h, int32_t Z)
{
    uint64_t x = 1469598103934665603ull;
    auto mix = [&x](uint64_t v) {
        for (int b = 0; b < 8; ++b) {
            x ^= (v >> (8 * b)) & 0xffu;
            x *= 1099511628211ull;
        }
    };
    mix(static_cast<uint64_t>(h.m));
    mix(static_cast<uint64_t>(h.n));
    mix(static_cast<uint64_t>(h.col_idx.size()));
    mix(static_cast<uint64_t>(Z));
    std::vector<int64_t> rows(h.max_row_deg + 1, 0), cols(h.max_col_deg + 1, 0);
    for (int32_t i = 0; i < h.m; ++i)
        rows[h.row_ptr[i + 1] - h.row_ptr[i]]++;
    for (int32_t j = 0; j < h.n; ++j)
        cols[h.col_ptr[j + 1] - h.col_ptr[j]]++;
    for (int64_t v : rows)
        mix(static_cast<uint64_t>(v));
    mix(~0ull);
    for (int64_t v : cols)
        mix(static_cast<uint64_t>(v));
    return x;
}

// Host image of the device allocation.  Tables are sized before they are
// filled: a code's handle is made once, but a program waits for it.
struct TableImage {
    std::vector<int32_t> words;
    // `count` words of `fill` on a 16-byte boundary (quads are 16-byte loads).
    size_t take(size_t count, int32_t fill)
    {
        const size_t at = (words.size() + 3) / 4 * 4;
        words.resize(at, 0);
        words.resize(at + count, fill);
        return at;
    }
};

constexpr int64_t kLdsBytes = 160 * 1024;  // one workgroup's, gfx950

// Splits of a row of degree d: halves, or (layered) quarters.
void part_span(int32_t d, int part, int parts, int32_t &k0, int32_t &len)
{
    const int32_t h = (d + 1) / 2, q1 = (h + 1) / 2, q3 = h + (d - h + 1) / 2;
    const int32_t cut2[3] = {0, h, d}, cut4[5] = {0, q1, h, q3, d};
    const int32_t *cut = parts == 2 ? cut2 : cut4;
    k0 = cut[part];
    len = cut[part + 1] - cut[part];
}

struct FusedOffsets {
    bool built = false, explicit_too = false;
    int32_t row_groups = 0, slot_words = 0;
    int32_t row_words = 0, col_words = 0, lay_words = 0;
    size_t row_grp = 0, row_tab = 0, col_grp = 0, col_tab = 0;
    size_t row_grp_x = 0, row_tab_x = 0, row_pos_x = 0, col_tab_x = 0;
    size_t lay_ptr = 0, lay_grp = 0, lay_tab = 0;
};

// The tables described at FusedTables, appended to `im`.  Codes whose messages
// cannot fit a workgroup in FP32, or whose rows are longer than the kernel's
// bodies, get none.
FusedOffsets fused_tables(const HostLayout &h, const std::vector<int32_t> &layer_ptr, TableImage &im)
{
    FusedOffsets o;
    const int64_t E = static_cast<int64_t>(h.col_idx.size());
    if (h.max_row_deg > 32 || 4 * (E + h.n) > kLdsBytes)
        return o;
    o.built = true;
    const int32_t first = ldpc::fused_first_message(h.n), inf = 4 * h.n, minus_zero = 4 * (h.n + 1),
                  junk = 4 * (h.n + 2);
    auto degree = [&](int32_t i) { return h.row_ptr[i + 1] - h.row_ptr[i]; };
    // rows by descending degree, stable; `filled` of them have an edge
    std::vector<int32_t> order(h.m), rank(34, 0);
    for (int32_t i = 0; i < h.m; ++i)
        ++rank[33 - degree(i)];
    for (int32_t d = 1; d < 34; ++d)
        rank[d] += rank[d - 1];
    const int32_t filled = rank[32];
    for (int32_t i = h.m - 1; i >= 0; --i)
        order[--rank[33 - degree(i)]] = i;
    o.row_groups = (filled + 31) / 32;

    std::vector<int32_t> slot_of(E);  // padded order: an edge's word among the messages
    auto rows = [&](bool x, size_t &grp_at, size_t &tab_at, size_t *pos_at) {
        size_t quad_rows = 0;
        for (int32_t g = 0; g < o.row_groups; ++g)
            quad_rows += x ? 4 : ((degree(order[32 * g]) + 1) / 2 + 3) / 4;
        grp_at = im.take(2 * static_cast<size_t>(o.row_groups), 0);
        tab_at = im.take(quad_rows * 256, inf);
        if (!x)
            o.row_words = static_cast<int32_t>(quad_rows * 256);
        if (x)
            *pos_at = im.take(quad_rows * 256, junk);
        int32_t *grp = im.words.data() + grp_at, *tab = im.words.data() + tab_at;
        int32_t *pos = x ? im.words.data() + *pos_at : nullptr;
        int32_t slots = 0, quad_row = 0;
        for (int32_t g = 0; g < o.row_groups; ++g) {
            const int32_t longest = (degree(order[32 * g]) + 1) / 2;
            grp[2 * g] = longest << 16 | slots;
            grp[2 * g + 1] = quad_row;
            for (int32_t lane = 0; lane < 64; ++lane) {
                const int32_t sr = 32 * g + (lane & 31);
                if (sr >= filled)
                    continue;
                int32_t k0, len;
                part_span(degree(order[sr]), lane >> 5, 2, k0, len);
                const int32_t e0 = h.row_ptr[order[sr]] + k0;
                const size_t base = static_cast<size_t>(quad_row) * 256 + static_cast<size_t>(lane) * 4;
                for (int32_t k = 0; k < len; ++k) {
                    const size_t at = base + static_cast<size_t>(k >> 2) * 256 + (k & 3);
                    tab[at] = 4 * h.col_idx[e0 + k];
                    if (x)
                        pos[at] = 4 * (first + e0 + k);
                    else
                        slot_of[e0 + k] = (slots + k) * 64 + lane;
                }
            }
            slots += longest;
            quad_row += x ? 4 : (longest + 3) / 4;
        }
        return slots * 64;
    };
    auto columns = [&](bool x, size_t *grp_at, size_t &tab_at) {
        const int32_t groups = (h.n + 63) / 64;
        std::vector<int32_t> longest(groups, 0);
        size_t quad_rows = 0;
        for (int32_t g = 0; g < groups; ++g) {
            for (int32_t j = 64 * g; j < std::min(h.n, 64 * g + 64); ++j)
                longest[g] = std::max(longest[g], h.col_ptr[j + 1] - h.col_ptr[j]);
            quad_rows += (longest[g] + 3) / 4;
        }
        if (grp_at)
            *grp_at = im.take(2 * static_cast<size_t>(groups), 0);
        tab_at = im.take(quad_rows * 256, minus_zero);
        if (!x)
            o.col_words = static_cast<int32_t>(quad_rows * 256);
        int32_t *grp = grp_at ? im.words.data() + *grp_at : nullptr, *tab = im.words.data() + tab_at;
        int32_t quad_row = 0;
        for (int32_t g = 0; g < groups; ++g) {
            if (grp) {
                grp[2 * g] = longest[g];
                grp[2 * g + 1] = quad_row;
            }
            for (int32_t j = 64 * g; j < std::min(h.n, 64 * g + 64); ++j) {
                const int32_t *edge = h.col_edge.data() + h.col_ptr[j];
                const size_t base = static_cast<size_t>(quad_row) * 256 + static_cast<size_t>(j & 63) * 4;
                for (int32_t k = 0; k < h.col_ptr[j + 1] - h.col_ptr[j]; ++k)
                    tab[base + static_cast<size_t>(k >> 2) * 256 + (k & 3)] =
                        4 * (first + (x ? edge[k] : slot_of[edge[k]]));
            }
            quad_row += (longest[g] + 3) / 4;
        }
    };
    o.slot_words = rows(false, o.row_grp, o.row_tab, nullptr);
    columns(false, &o.col_grp, o.col_tab);
    // a type whose frames fit in CSR order but not in the padded order
    for (const int64_t ts : {4, 8})
        o.explicit_too |= ts * (first + o.slot_words) + 32 > kLdsBytes && ts * (first + E) <= kLdsBytes;
    if (o.explicit_too) {
        rows(true, o.row_grp_x, o.row_tab_x, &o.row_pos_x);
        columns(true, nullptr, o.col_tab_x);
    }

    auto longest_quarter = [&](int32_t r0, int32_t rows16) {
        int32_t longest = 0;
        for (int32_t r = r0; r < r0 + rows16; ++r)
            longest = std::max(longest, ((degree(r) + 1) / 2 + 1) / 2);
        return longest;
    };
    const size_t layers = layer_ptr.size() - 1;
    size_t groups = 0, words = 0;
    for (size_t l = 0; l < layers; ++l)
        for (int32_t r0 = layer_ptr[l]; r0 < layer_ptr[l + 1]; r0 += 16) {
            const int32_t rows16 = std::min(16, layer_ptr[l + 1] - r0);
            words += static_cast<size_t>((longest_quarter(r0, rows16) + 3) / 4) * 32 * rows16;
            ++groups;
        }
    o.lay_ptr = im.take(layers + 1, 0);
    o.lay_grp = im.take(2 * groups, 0);
    o.lay_tab = im.take(words, inf);
    o.lay_words = static_cast<int32_t>(words);
    int32_t *ptr = im.words.data() + o.lay_ptr, *grp = im.words.data() + o.lay_grp;
    int32_t *tab = im.words.data() + o.lay_tab;
    size_t g = 0, base = 0;
    for (size_t l = 0; l < layers; ++l) {
        ptr[l] = static_cast<int32_t>(g);
        for (int32_t r0 = layer_ptr[l]; r0 < layer_ptr[l + 1]; r0 += 16, ++g) {
            const int32_t rows16 = std::min(16, layer_ptr[l + 1] - r0), longest = longest_quarter(r0, rows16);
            const size_t half = static_cast<size_t>((longest + 3) / 4) * 16 * rows16;
            grp[2 * g] = longest << 8 | rows16;
            grp[2 * g + 1] = static_cast<int32_t>(base / 4);
            std::fill(tab + base + half, tab + base + 2 * half, junk);
            for (int32_t r = 0; r < rows16; ++r)
                for (int part = 0; part < 4; ++part) {
                    int32_t k0, len;
                    part_span(degree(r0 + r), part, 4, k0, len);
                    const int32_t e0 = h.row_ptr[r0 + r] + k0;
                    for (int32_t k = 0; k < len; ++k) {
                        const size_t at = base + (static_cast<size_t>(k >> 2) * 4 * rows16 + part * rows16 + r) * 4 +
                                          (k & 3);
                        tab[at] = 4 * h.col_idx[e0 + k];
                        tab[at + half] = 4 * (first + e0 + k);
                    }
                }
            base += 2 * half;
        }
    }
    ptr[layers] = static_cast<int32_t>(g);
    return o;
}

ldpc_status upload(const HostLayout &h, int32_t Z, ldpc_code_s *c)
{
    layer_tables(h, c->layer_ptr, c->layer_dmax);
    for (size_t l = 0; l + 1 < c->layer_ptr.size(); ++l)
        c->layer_rows = std::max(c->layer_rows, c->layer_ptr[l + 1] - c->layer_ptr[l]);
    TableImage im;
    im.words.reserve(10 * h.col_idx.size() + 4 * h.row_ptr.size() + 4 * h.col_ptr.size() + 4096);
    const FusedOffsets fo = fused_tables(h, c->layer_ptr, im);
    auto put = [&](const std::vector<int32_t> &v) {
        const size_t off = im.words.size();
        im.words.insert(im.words.end(), v.begin(), v.end());
        return off;
    };
    const size_t o_rp = put(h.row_ptr), o_ci = put(h.col_idx), o_cp = put(h.col_ptr), o_ce = put(h.col_edge);
    void *d = nullptr;
    if (hipMalloc(&d, std::max<size_t>(im.words.size(), 1) * sizeof(int32_t)) != hipSuccess)
        return LDPC_ENOMEM;
    if (hipMemcpy(d, im.words.data(), im.words.size() * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess) {
        (void)hipFree(d);
        return LDPC_EDEVICE;
    }
    const int32_t *base = static_cast<const int32_t *>(d);
    c->d_mem = d;
    c->row_ptr = base + o_rp;
    c->col_idx = base + o_ci;
    c->col_ptr = base + o_cp;
    c->col_edge = base + o_ce;
    if (fo.built) {
        ldpc::FusedTables &t = c->fused;
        t.row_groups = fo.row_groups;
        t.slot_words = fo.slot_words;
        t.row_words = fo.row_words;
        t.col_words = fo.col_words;
        t.lay_words = fo.lay_words;
        t.row_grp = base + fo.row_grp;
        t.row_tab = base + fo.row_tab;
        t.col_grp = base + fo.col_grp;
        t.col_tab = base + fo.col_tab;
        if (fo.explicit_too) {
            t.row_grp_x = base + fo.row_grp_x;
            t.row_tab_x = base + fo.row_tab_x;
            t.row_pos_x = base + fo.row_pos_x;
            t.col_tab_x = base + fo.col_tab_x;
        }
        t.lay_ptr = base + fo.lay_ptr;
        t.lay_grp = base + fo.lay_grp;
        t.lay_tab = base + fo.lay_tab;
    }
    c->m = h.m;
    c->n = h.n;
    c->E = static_cast<int64_t>(h.col_idx.size());
    c->max_row_deg = h.max_row_deg;
    c->max_col_deg = h.max_col_deg;
    for (int32_t j = 0; j < h.n; ++j) {
        const int64_t d = h.col_ptr[j + 1] - h.col_ptr[j];
        c->column_reads += d * d;
    }
    c->shape_hash = shape_hash(h, Z);
    return LDPC_OK;
}

}  // namespace

bool ldpc::code_on_current_device(const ldpc_code_s *c)
{
    int dev = -1;
    return hipGetDevice(&dev) == hipSuccess && dev == c->device;
}

extern "C" const char *ldpc_status_str(ldpc_status s)
{
    switch (s) {
    case LDPC_OK: return "ok";
    case LDPC_EINVAL: return "invalid argument";
    case LDPC_ENOMEM: return "out of memory";
    case LDPC_EDEVICE: return "HIP runtime error";
    case LDPC_EBUSY: return "busy";
    case LDPC_EUNSUPPORTED: return "unsupported";
    }
    return "unknown status";
}

extern "C" ldpc_status ldpc_code_from_csr(int32_t m, int32_t n, const int32_t *row_ptr, const int32_t *col_idx,
                                          ldpc_code *out)
try {
    if (!out)
        return LDPC_EINVAL;
    HostLayout h;
    ldpc_status st = build_host_layout(m, n, row_ptr, col_idx, h);
    if (st != LDPC_OK)
        return st;
    auto *c = new (std::nothrow) ldpc_code_s();
    if (!c)
        return LDPC_ENOMEM;
    if (hipGetDevice(&c->device) != hipSuccess) {
        delete c;
        return LDPC_EDEVICE;
    }
    st = upload(h, 0, c);
    if (st != LDPC_OK) {
        delete c;
        return st;
    }
    *out = c;
    return LDPC_OK;
} catch (...) {
    return ldpc::status_of_exception();
}

extern "C" ldpc_status ldpc_code_from_qc(int32_t mb, int32_t nb, int32_t Z, const int32_t *shifts, ldpc_code *out)
try {
    if (!out || !shifts || mb < 1 || nb < 1 || Z < 1)
        return LDPC_EINVAL;
    if (static_cast<int64_t>(mb) * Z > INT32_MAX / 2 || static_cast<int64_t>(nb) * Z > INT32_MAX / 2)
        return LDPC_EUNSUPPORTED;
    for (int64_t k = 0; k < static_cast<int64_t>(mb) * nb; ++k)
        if (shifts[k] < -1 || shifts[k] >= Z)
            return LDPC_EINVAL;
    // CSR of the lifted matrix: row i*Z + r has, for each non-empty block
    // (i, j) in ascending j, the column j*Z + (r + s) mod Z.
    const int32_t m = mb * Z, n = nb * Z;
    std::vector<int32_t> row_ptr(m + 1, 0), col_idx;
    std::vector<int32_t> row_blk_start(mb + 1, 0), blk_col, blk_shift;
    for (int32_t i = 0; i < mb; ++i) {
        for (int32_t j = 0; j < nb; ++j)
            if (shifts[i * nb + j] >= 0) {
                blk_col.push_back(j);
                blk_shift.push_back(shifts[i * nb + j]);
            }
        row_blk_start[i + 1] = static_cast<int32_t>(blk_col.size());
    }
    const int32_t nblocks = static_cast<int32_t>(blk_col.size());
    col_idx.reserve(static_cast<size_t>(nblocks) * Z);
    for (int32_t i = 0; i < mb; ++i)
        for (int32_t r = 0; r < Z; ++r) {
            for (int32_t b = row_blk_start[i]; b < row_blk_start[i + 1]; ++b)
                col_idx.push_back(blk_col[b] * Z + (r + blk_shift[b]) % Z);
            row_ptr[i * Z + r + 1] = static_cast<int32_t>(col_idx.size());
        }
    HostLayout h;
    ldpc_status st = build_host_layout(m, n, row_ptr.data(), col_idx.data(), h);
    if (st != LDPC_OK)
        return st;
    auto *c = new (std::nothrow) ldpc_code_s();
    if (!c)
        return LDPC_ENOMEM;
    if (hipGetDevice(&c->device) != hipSuccess) {
        delete c;
        return LDPC_EDEVICE;
    }
    st = upload(h, Z, c);
    if (st != LDPC_OK) {
        delete c;
        return st;
    }
    c->is_qc = true;
    c->mb = mb;
    c->Z = Z;
    c->nblocks = nblocks;
    c->qc_words = (mb + 1) + 3 * nblocks + (nb + 1);
    *out = c;
    return LDPC_OK;
} catch (...) {
    return ldpc::status_of_exception();
}

extern "C" ldpc_status ldpc_code_info(ldpc_code code, int32_t *m, int32_t *n, int64_t *edges)
try {
    if (!code)
        return LDPC_EINVAL;
    if (m)
        *m = code->m;
    if (n)
        *n = code->n;
    if (edges)
        *edges = code->E;
    return LDPC_OK;
} catch (...) {
    return ldpc::status_of_exception();
}

extern "C" ldpc_status ldpc_code_layers(ldpc_code code, int32_t *nlayers, int32_t *min_rows, int32_t *max_rows)
try {
    if (!code)
        return LDPC_EINVAL;
    const int32_t L = static_cast<int32_t>(code->layer_dmax.size());
    int32_t lo = L ? INT32_MAX : 0, hi = 0;
    for (int32_t l = 0; l < L; ++l) {
        const int32_t r = code->layer_ptr[l + 1] - code->layer_ptr[l];
        lo = std::min(lo, r);
        hi = std::max(hi, r);
    }
    if (nlayers)
        *nlayers = L;
    if (min_rows)
        *min_rows = lo;
    if (max_rows)
        *max_rows = hi;
    return LDPC_OK;
} catch (...) {
    return ldpc::status_of_exception();
}

extern "C" void ldpc_code_destroy(ldpc_code code)
try {
    if (!code)
        return;
    if (code->d_mem) {
        int prev = -1;
        (void)hipGetDevice(&prev);
        (void)hipSetDevice(code->device);
        (void)hipFree(code->d_mem);
        if (prev >= 0)
            (void)hipSetDevice(prev);
    }
    delete code;
} catch (...) {
}

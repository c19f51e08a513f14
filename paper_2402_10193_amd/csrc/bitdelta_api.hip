// C ABI of the library (include/bitdelta.h): argument checks, token grouping, kernel choice.
// Everything here runs on the host; nothing is enqueued before the arguments have passed.
#include "bitdelta.h"

#include <algorithm>
#include <cstring>
#include <utility>
#include <vector>

#include "bd_launch.h"
#include "bd_tiled.h"

namespace {

using bd::DecodeMeta;
using bd::kMaxDecodeTokens;

constexpr int kVersion = 223;   // 0.2.23
constexpr int kVariantRowWave = 1;
constexpr int kVariantRowMajorMfma = 2;   // the matrix-core decode kernel on the row-major tensors (in % 128 == 0)
constexpr int kVariantPrefillSmall = 4;   // T > 32 with a workspace: the 128 x 128 tile GEMM
constexpr int kVariantPrefillBig = 5;     // ... the 128 x 256 tile GEMM (in % 64 == 0), one wavefront per SIMD
constexpr int kVariantPrefillBig8 = 6;    // ... the same tile with two wavefronts per SIMD
constexpr int kVariantPrefillBigWhole = 7;   // ... as 5, but never cutting the tiles of the last round in two
constexpr int kVariantPrefillMerged = 8;     // ... one product on W + alpha S, formed in fp16 on the way to the matrix cores (256 x 256 tiles)
constexpr int kVariantWide = 10;             // the kernel for tens to a few hundred tokens; 16 R + n: R row blocks and up to n column tiles per workgroup
constexpr int kVariantPanels = 128;          // panels, row-major; + n: up to n column tiles per workgroup

inline bool misaligned(const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) != 0; }

inline bool overlaps(const void* a, size_t abytes, const void* b, size_t bbytes) {
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + bbytes && b0 < a0 + abytes;
}

// Tokens [t0, t0 + n) of the call -> one launch's bookkeeping: columns sorted by tenant
// (stable), jobs = runs of equal tenant cut at the 16-column tile boundary.
void build_meta(const int32_t* tenant_of_token, int64_t t0, int n, DecodeMeta* m) {
    std::memset(m, 0, sizeof(*m));
    m->T = n;
    int order[kMaxDecodeTokens];
    for (int i = 0; i < n; ++i) {
        order[i] = i;
        m->tenant_of_token[i] = tenant_of_token[t0 + i];
    }
    std::stable_sort(order, order + n, [&](int a, int b) { return m->tenant_of_token[a] < m->tenant_of_token[b]; });
    int jobs = 0;
    for (int col = 0; col < n; ++col) {
        const int tok = order[col];
        const int tenant = m->tenant_of_token[tok];
        m->token_of_col[col] = (int32_t)tok;
        m->tenant_of_col[col] = tenant;
        const int tile = col >> 4, cin = col & 15;
        if (jobs > 0 && m->job_tenant[jobs - 1] == tenant && m->job_tile[jobs - 1] == tile) {
            m->job_col_end[jobs - 1] = (int32_t)(cin + 1);
        } else {
            m->job_tenant[jobs] = tenant;
            m->job_tile[jobs] = (int32_t)tile;
            m->job_col_begin[jobs] = (int32_t)cin;
            m->job_col_end[jobs] = (int32_t)(cin + 1);
            ++jobs;
        }
    }
    m->n_jobs = jobs;
    for (int tile = 0; tile < 2; ++tile) {
        int b = 0;
        while (b < jobs && m->job_tile[b] < tile) ++b;
        int e = b;
        while (e < jobs && m->job_tile[e] == tile) ++e;
        m->tile_job_begin[tile] = b;
        m->tile_job_end[tile] = e;
        for (int sl = 0; sl < 16; ++sl) {
            const bool real = b + sl < e;
            m->slot_tenant[tile][sl] = real ? m->job_tenant[b + sl] : (b < e ? m->job_tenant[b] : 0);
            m->slot_col_begin[tile][sl] = real ? m->job_col_begin[b + sl] : 0;
            m->slot_col_end[tile][sl] = real ? m->job_col_end[b + sl] : 0;
        }
    }
}

bd_status check_linear_args(const void* x, const void* w, const void* packed_by_tenant, const void* alpha_by_tenant,
                            const int32_t* tenant_of_token, const void* y, int64_t T, int64_t out, int64_t in,
                            int32_t n_tenants, size_t w_bytes_per_el = 2) {
    if (T < 0 || out < 0 || in < 0 || n_tenants < 0 || T > 65535) return BD_ERR_SHAPE;
    if (in % 32 != 0) return BD_ERR_SHAPE;
    if (out > (int64_t)1 << 31 || in > (int64_t)1 << 31) return BD_ERR_SHAPE;
    if (T == 0 || out == 0) return BD_OK;
    if (!x || !w || !packed_by_tenant || !alpha_by_tenant || !tenant_of_token || !y) return BD_ERR_NULL;
    if (misaligned(x, 16) || misaligned(w, 16) || misaligned(y, 16) || misaligned(packed_by_tenant, 8) ||
        misaligned(alpha_by_tenant, 4))
        return BD_ERR_ALIGN;
    for (int64_t t = 0; t < T; ++t)
        if (tenant_of_token[t] < 0 || tenant_of_token[t] >= n_tenants) return BD_ERR_TENANT;
    const size_t ybytes = (size_t)T * out * 2;
    if (overlaps(y, ybytes, x, (size_t)T * in * 2) || overlaps(y, ybytes, w, (size_t)out * in * w_bytes_per_el)) return BD_ERR_ALIAS;
    return BD_OK;
}

// Prefill (T > 32): the token permutation and the tenant of every 128-row tile live in the workspace.
// At most ceil(T / 128) full tiles plus one ragged tile per tenant that has a token.
size_t prefill_table_bytes(int64_t T, int32_t n_tenants, bool merged_too = false);
size_t prefill_workspace_bytes(int64_t T, int32_t n_tenants) {
    if (T <= kMaxDecodeTokens || n_tenants < 0) return 0;
    return prefill_table_bytes(T, n_tenants, true);
}
size_t tiled_gemm_workspace_bytes(int64_t T, int32_t n_tenants);
// The token tables of the GEMM: tiles of 128 rows (merged_too: or of the 256 rows of the one-product form, whichever
// table is larger); every tenant with a token ends in one partly filled tile at most.
size_t prefill_table_bytes(int64_t T, int32_t n_tenants, bool merged_too) {
    if (T < 1 || n_tenants < 0) return 0;
    size_t bytes = 0;
    for (const int64_t rows : {(int64_t)bd::kPrefillTile, (int64_t)bd::kPrefillMergedTile}) {
        if (rows != bd::kPrefillTile && !merged_too) continue;
        const int64_t tiles = (T + rows - 1) / rows + std::min<int64_t>(n_tenants, T);
        bytes = std::max(bytes, (size_t)tiles * (size_t)(rows + 1) * sizeof(int32_t));
    }
    return (bytes + 255) & ~(size_t)255;
}

// bd_linear_multitenant_tiled_gemm: the token tables and, behind them, the table of the tenants' sign pointers
size_t tiled_gemm_workspace_bytes(int64_t T, int32_t n_tenants) {
    const size_t tables = prefill_table_bytes(T, n_tenants, true);
    if (tables == 0) return 0;
    return tables + (((size_t)n_tenants * 8 + 8 + 255) & ~(size_t)255);
}

// Token ids by tenant, tokens of one tenant in their order.  (Tenant ids have been checked.)
std::vector<int32_t> order_by_tenant(const int32_t* tenant_of_token, int64_t T, int32_t n_tenants) {
    std::vector<int32_t> order((size_t)T);
    if (std::is_sorted(tenant_of_token, tenant_of_token + T)) {
        for (int64_t i = 0; i < T; ++i) order[(size_t)i] = (int32_t)i;
    } else if (n_tenants <= 8 * T) {
        std::vector<int32_t> next((size_t)n_tenants + 1, 0);
        for (int64_t i = 0; i < T; ++i) ++next[(size_t)tenant_of_token[i] + 1];
        for (int32_t t = 0; t < n_tenants; ++t) next[(size_t)t + 1] += next[(size_t)t];
        for (int64_t i = 0; i < T; ++i) order[(size_t)next[(size_t)tenant_of_token[i]]++] = (int32_t)i;
    } else {   // a table of counts would be larger than the batch
        for (int64_t i = 0; i < T; ++i) order[(size_t)i] = (int32_t)i;
        std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return tenant_of_token[a] < tenant_of_token[b]; });
    }
    return order;
}

int cus_or_256() {
    int cus = 256;
    if (bd::device_cu_count(&cus) != hipSuccess || cus < 1) cus = 256;
    return cus;
}

// Cuts the tokens (`order`: sorted by tenant) into tiles of 128 rows (merged: 256) that never mix tenants, writes
// the two tables into the workspace (through kernel arguments: no host-to-device copy call) and runs the GEMM.
// k_planes = 0: one plane per tenant; 1..8: tables indexed by tenant * k_planes + plane.  wscale: the 8-bit base's row
// scales (w is then the int8 tensor).  big_waves = 0: the 128 x 128 tiles.
hipError_t run_prefill(const uint16_t* x, const void* w, const uint32_t* const* packed_by_tenant,
                       const float* alpha_by_tenant, const int32_t* tenant_of_token, const std::vector<int32_t>& order, uint16_t* y, int64_t T, int64_t out,
                       int64_t in, void* workspace, hipStream_t st, int big_waves, bool halve_last_round,
                       int k_planes = 0, const float* wscale = nullptr, bool merged = false,
                       const uint32_t* const* tiled_by_tenant_host = nullptr, int32_t n_tenants = 0) {
    const int64_t tile_rows = merged ? bd::kPrefillMergedTile : bd::kPrefillTile;
    // The tiles: (first token of the sorted order, rows).  Where they fill the compute units more than once, those with more than
    // half a tile of rows run first and the launch ends with short ones (with an eighth of either kind for every XCD: 1100 tokens of
    // 13 tenants on 11008 x 4096 264 -> 232 us, as one product 269 -> 229; 3000 of 12 on 4096 x 4096 189 -> 162).  Tiles that all run
    // at once stay in the tenants' order: sorted, an XCD would run the same N tiles less often side by side (512 tokens of
    // 8 tenants on 4096 x 4096: 57 us as they come, 65 sorted).
    std::vector<std::pair<int64_t, int64_t>> tiles, short_tiles;
    int64_t n_tiles = 0;
    for (int64_t i = 0, n = 0; i < T; ++i, ++n)
        if (i == 0 || n == tile_rows || tenant_of_token[order[(size_t)i]] != tenant_of_token[order[(size_t)i - 1]]) {
            ++n_tiles;
            n = 0;
        }
    const bool long_first = n_tiles * ((out + 255) / 256) > (int64_t)cus_or_256();
    for (int64_t i = 0; i < T;) {
        const int32_t tenant = tenant_of_token[order[(size_t)i]];
        int64_t e = i;
        while (e < T && tenant_of_token[order[(size_t)e]] == tenant) ++e;
        for (int64_t t0 = i; t0 < e; t0 += tile_rows)
            (2 * std::min(tile_rows, e - t0) > tile_rows || !long_first ? tiles : short_tiles).emplace_back(t0, std::min(tile_rows, e - t0));
        i = e;
    }
    const int n_large = (int)tiles.size();
    tiles.insert(tiles.end(), short_tiles.begin(), short_tiles.end());
    std::vector<int32_t> row_token, tile_tenant;
    row_token.reserve(tiles.size() * (size_t)tile_rows);
    for (const auto& [t0, rows] : tiles) {
        tile_tenant.push_back(tenant_of_token[order[(size_t)t0]]);
        row_token.insert(row_token.end(), order.begin() + t0, order.begin() + t0 + rows);
        row_token.insert(row_token.end(), (size_t)(tile_rows - rows), -1);
    }
    const int n_mtiles = (int)tile_tenant.size();
    std::vector<int32_t> all(row_token);
    all.insert(all.end(), tile_tenant.begin(), tile_tenant.end());
    // Serving layout: the tenants' sign pointers come as a host array; the GEMM reads them from a device table, which
    // travels behind the token tables (8-byte aligned).
    const bool tiled = tiled_by_tenant_host != nullptr;
    size_t pointer_table_at = 0;
    if (tiled) {
        if (all.size() & 1) all.push_back(0);
        pointer_table_at = all.size();
        for (int32_t t = 0; t < n_tenants; ++t) {
            const uint64_t p = (uint64_t)(uintptr_t)tiled_by_tenant_host[t];
            all.push_back((int32_t)(uint32_t)p);
            all.push_back((int32_t)(uint32_t)(p >> 32));
        }
    }
    int32_t* dst = (int32_t*)workspace;
    // The tables as runs of values that count up or repeat (tokens that arrive grouped by tenant: a few runs for the
    // whole batch), where that takes fewer launches than the values themselves.
    std::vector<int32_t> runs;   // triples: first index, first value, n (> 0 counting up, < 0 repeated)
    for (size_t i = 0; i < all.size();) {
        size_t e = i + 1;
        const int32_t step = e < all.size() ? all[e] - all[i] : 0;
        if (step == 0 || step == 1)
            while (e < all.size() && all[e] - all[e - 1] == step) ++e;
        runs.insert(runs.end(), {(int32_t)i, all[i], step == 1 ? (int32_t)(e - i) : -(int32_t)(e - i)});
        i = e;
    }
    if ((runs.size() / 3 + 319) / 320 < (all.size() + 959) / 960) {
        for (size_t off = 0; off < runs.size(); off += 960) {
            bd::PrefillMetaChunk c;
            const int n = (int)std::min<size_t>(960, runs.size() - off);
            std::memcpy(c.v, runs.data() + off, (size_t)n * sizeof(int32_t));
            const hipError_t e = bd::launch_prefill_meta_runs(c, dst, n / 3, st);
            if (e != hipSuccess) return e;
        }
    } else {
        for (size_t off = 0; off < all.size(); off += 960) {
            bd::PrefillMetaChunk c;
            const int n = (int)std::min<size_t>(960, all.size() - off);
            std::memcpy(c.v, all.data() + off, (size_t)n * sizeof(int32_t));
            const hipError_t e = bd::launch_prefill_meta(c, dst + off, n, st);
            if (e != hipSuccess) return e;
        }
    }
    if (tiled) packed_by_tenant = (const uint32_t* const*)(dst + pointer_table_at);
    if (merged)
        return bd::launch_linear_prefill_merged(x, (const uint16_t*)w, packed_by_tenant, alpha_by_tenant, dst,
                                                dst + row_token.size(), n_mtiles, n_large, y, T, out, in, halve_last_round, tiled, st);
    if (big_waves)
        return bd::launch_linear_prefill_big(x, w, packed_by_tenant, alpha_by_tenant, wscale, dst, dst + row_token.size(), n_mtiles, n_large, y, T,
                                             out, in, big_waves, halve_last_round, tiled, st);
    if (tiled) return hipErrorInvalidValue;   // the 128 x 128 tiles read the row-major tensors only
    return bd::launch_linear_prefill(x, w, packed_by_tenant, alpha_by_tenant, wscale, dst, dst + row_token.size(), n_mtiles, n_large, y,
                                     out, in, k_planes, st);
}

// ---- batches between a decode launch and a GEMM: linear_wide.hip ----

// Column tiles of one call: each tenant's tokens cut into tiles of 16 columns.
struct WideTiles {
    std::vector<int32_t> tenant;               // per tile
    std::vector<uint16_t> token;               // 16 per tile, kWideNoToken where empty
    int64_t tokens = 0;
};
WideTiles wide_tiles(const int32_t* tenant_of_token, const std::vector<int32_t>& order) {
    WideTiles t;
    t.tokens = (int64_t)order.size();
    int in_tile = 16;
    for (size_t i = 0; i < order.size(); ++i) {
        const int32_t tenant = tenant_of_token[order[i]];
        if (in_tile == 16 || tenant != t.tenant.back()) {
            t.tenant.push_back(tenant);
            t.token.insert(t.token.end(), 16, (uint16_t)bd::kWideNoToken);
            in_tile = 0;
        }
        t.token[(t.tenant.size() - 1) * 16 + (size_t)in_tile++] = (uint16_t)order[i];
    }
    return t;
}

// What the time of eight wavefronts goes by that have u[w] steps each, two to a SIMD, issuing in turn: between the longest
// wavefront and half the longest pair (a third and two thirds, fitted).
double steps_of_waves(const int (&u)[8]) {
    int longest = 0, pair = 0;
    for (int w = 0; w < 4; ++w) {
        longest = std::max({longest, u[w], u[w + 4]});
        pair = std::max(pair, u[w] + u[w + 4]);
    }
    return (longest + pair) / 3.0;
}
// Units (128 of `in`) of the wavefronts of a workgroup of the wide kernel
double wide_units(int64_t in, bool rowmajor) {
    const int units = (int)(in / 128), KT = (int)bd::tiled_k_tiles(in), nw = bd::wide_k_waves(KT), subs = 8 / nw;
    int u[8];
    for (int w = 0; w < 8; ++w)
        u[w] = rowmajor ? (units - w + 7) / 8 : std::min(2 * ((w / subs + 1) * KT / nw), units) - 2 * (w / subs * KT / nw);
    return steps_of_waves(u);
}

struct WidePlan {
    int R, per_chunk;
    double us;
};

// The panel kernel on n column tiles (row-major): one workgroup per compute unit at a time, some 4 us around its loop, and per iteration and column
// tile 0.31 us (8-bit base 0.29, k planes 0.03 + 0.18 k).  Fitted to 90 batches of 33 to 700 tokens on 300 .. 12000 x 512 .. 11520 (fp16, one plane) and
// to 100 of 24 to 4096 tokens on 500 .. 11008 x 512 .. 11008 (50 over the 8-bit base, 50 with 2 to 4 planes) with every chunk size: 8 % at the 10 % and
// 90 % quantiles; the chunk it picks is the quickest in all but a few.
WidePlan panel_plan(int n, int64_t out, int64_t in, int cus, int planes, bool q8) {
    WidePlan best{0, 0, 1e30};
    const int64_t groups = (bd::tiled_row_blocks(out) + bd::kPanelRowBlocks - 1) / bd::kPanelRowBlocks, iterations = ((in + 127) / 128 + 1) / 2;
    const int64_t per_xcd = std::max(1, cus / 8);
    const double fixed = q8 ? 4.1 : planes == 1 ? 3.4 : 3.8, tile = q8 ? 0.29 : planes == 1 ? 0.306 : 0.03 + 0.183 * planes;
    for (int run = 2; run <= bd::panel_max_chunk(planes); ++run) {
        const int chunks = (n + run - 1) / run;
        const int64_t rounds = ((groups + 7) / 8 * chunks + per_xcd - 1) / per_xcd;
        const double us = (double)rounds * (fixed + tile * (double)(iterations * run)) + (double)chunks * (double)out * (double)in * (q8 ? 0.065e-6 : 0.075e-6);
        if (us < best.us) best = WidePlan{bd::kPanelRowBlocks, std::min(run, n), us};
    }
    return best;
}
// (No bound by the stream, nor in gemm_extended_us, which this is compared with: few tokens on matrices of a gigabyte come out below what HBM gives, but
// both ways then stream the same bytes.)
double panel_us(int n_all, int64_t out, int64_t in, int cus, int planes, bool q8) {
    double us = 3.5;
    const int launches = (n_all + bd::kWideMaxTiles - 1) / bd::kWideMaxTiles;
    for (int l = 0; l < launches; ++l)
        us += panel_plan((int)((int64_t)n_all * (l + 1) / launches - (int64_t)n_all * l / launches), out, in, cus, planes, q8).us;
    return us;
}
// What panels of any kind take: whole units or one half unit at the end of a row, 32-bit offsets, token ids below the mark of an empty column
bool panel_fits(int64_t T, int64_t out, int64_t in, int planes, bool q8) {
    return planes >= 1 && planes <= bd::kPanelMaxPlanes && in >= 128 && in % 64 == 0 && out >= 1 && T < 65535 &&
           (uint64_t)T * (uint64_t)in * 2 < ((uint64_t)1 << 32) && (uint64_t)out * (uint64_t)in * (q8 ? 1 : 2) < ((uint64_t)1 << 32);
}

// How a launch of n column tiles is cut: row blocks per workgroup (1 or 2; kPanelRowBlocks: the panel kernel), column tiles per workgroup, and its
// estimated time: workgroups take turns on the compute units of their XCD (LDS allows one at a time, the row blocks are dealt to the XCDs), some 4 us
// around the loop of each, and every chunk fetches the base again.  Fitted to 3480 times: the batches described at BatchShape, every
// split.  10 % at the 10 % and 90 % quantiles; the split it picks is the quickest or within 7 % of it in 95 % of the batches.
WidePlan wide_plan(int n, int64_t tokens, int64_t out, int64_t in, int cus, bool rowmajor) {
    WidePlan best{0, 0, 1e30};
    const int64_t rb = bd::tiled_row_blocks(out), per_xcd = std::max(1, cus / 8);
    const double units = wide_units(in, rowmajor);
    for (int R = 1; R <= 2; ++R) {
        const int64_t per_group = R * (rowmajor ? 1 : 8 / bd::wide_k_waves((int)bd::tiled_k_tiles(in))), groups = (rb + per_group - 1) / per_group;
        for (int run = 2; run <= bd::wide_max_chunk(R, (int)bd::tiled_k_tiles(in), rowmajor); run += 2) {   // instantiated for even numbers
            const int chunks = (n + run - 1) / run;   // all but the last one full
            const int64_t rounds = ((groups + 7) / 8 * chunks + per_xcd - 1) / per_xcd;
            const double loop = units * (run - 1) * (rowmajor ? (R == 1 ? 0.52 : 0.79) : (R == 1 ? 0.48 : 0.69));
            const double us = (double)rounds * ((rowmajor ? 3.9 : 4.1) + loop) + (double)chunks * (double)out * (double)in * (rowmajor ? 0.15e-6 : 0.11e-6);
            if (us < best.us) best = WidePlan{R, std::min(run, n), us};
        }
    }
    // The panel kernel, row-major.  Where it lies against the others (us, the other ways' best / panel): 4096 x 4096 200 tokens of
    // 16 tenants 55 / 34, 11008 x 4096 500 of 32 285 / 220, 3278 x 1280 604 of 64 90 / 54; with few rows or one token per tenant the others win:
    // 996 x 7680 154 of 7 21 / 28, 330 x 2816 87 of 4 10 / 14, 6828 x 8320 58 of 51 241 / 324.
    // One group of panels per XCD, long rows, tiles of hardly more than one token: every wavefront's own fetch of x, what panels save, is then
    // mostly one line again and again.  460 x 9472 61 tokens of 53 34.5 / 35.7, 419 x 9344 57 of 52 34.5 / 35.7, 311 x 7552 44 of 43 26.4 / 27.1
    // (14 of 18 such batches); but 479 x 7680 195 of 34 31.2 / 29.9, 440 x 5632 36 of 34 21.3 / 20.9, 837 x 10112 58 of 45 49.9 / 50.3.
    if (rowmajor) {
        const WidePlan panel = panel_plan(n, out, in, cus, 1, false);
        if (panel.us < (out <= 512 && in > 7296 && tokens < 2 * (int64_t)n ? 0.95 : 1.0) * best.us) best = panel;
    }
    return best;
}
double wide_us(int n_all, int64_t tokens, int active, int64_t out, int64_t in, int cus, bool rowmajor) {
    double us = 3.0;
    const int launches = (n_all + bd::kWideMaxTiles - 1) / bd::kWideMaxTiles;
    for (int l = 0; l < launches; ++l)
        us += wide_plan((int)((int64_t)n_all * (l + 1) / launches - (int64_t)n_all * l / launches), tokens / launches, out, in, cus, rowmajor).us;
    const double elems = (double)out * (double)in;   // the stream: the base once, every active tenant's signs once
    return std::max(us, 6.0 + elems * (2.0 + (double)active / 8.0) / 4.5e6);
}

// The split that a variant number asks for: 0 = the plan's, kVariantPanels = the plan's of panels, -1 = none.
int panel_split_of_variant(int32_t variant, int planes) {
    return variant >= kVariantPanels && variant <= kVariantPanels + bd::panel_max_chunk(planes) ? variant : -1;
}
int wide_split_of_variant(int32_t variant, int64_t in, bool rowmajor) {
    if (variant == kVariantWide) return 0;
    if (rowmajor && variant >= kVariantPanels) return panel_split_of_variant(variant, 1);
    const int R = variant >> 4, n = variant & 15;
    return (R == 1 || R == 2) && n >= 1 && n <= bd::wide_max_chunk(R, (int)bd::tiled_k_tiles(in), rowmajor) ? variant : -1;
}

bool wide_fits(int64_t T, int64_t out, int64_t in) {
    return in >= 128 && in % 128 == 0 && out >= 1 && T < 65535 && (uint64_t)T * (uint64_t)in * 2 < ((uint64_t)1 << 32) &&
           (uint64_t)(bd::tiled_row_blocks(out) * bd::tiled_k_tiles(in)) * bd::kTileBaseBytes < ((uint64_t)1 << 32);
}

// packed_dev: the row-major tensors (device pointer table); otherwise w is the tiled base and tiled_host the tenants' tiled deltas.
// panel_planes > 0: panels, with that many planes per tenant (tables indexed by tenant * planes + plane) or, wscale given, the int8 base
hipError_t run_wide(const WideTiles& t, const uint16_t* x, const uint16_t* w, const uint32_t* const* packed_dev,
                    const uint32_t* const* tiled_host, const float* alpha, uint16_t* y, int64_t out, int64_t in, hipStream_t st,
                    int split = 0, int panel_planes = 0, const float* wscale = nullptr, bool inf_in_parts = false) {
    const int cus = cus_or_256(), n_all = (int)t.tenant.size(), launches = (n_all + bd::kWideMaxTiles - 1) / bd::kWideMaxTiles;
    for (int l = 0; l < launches; ++l) {
        const int first = (int)((int64_t)n_all * l / launches), n = (int)((int64_t)n_all * (l + 1) / launches) - first;
        bd::WideArgs a;
        std::memset(&a, 0, sizeof(a));
        a.x = x;
        a.w = w;
        a.y = y;
        a.packed_by_tenant = packed_dev;
        a.alpha_by_tenant = alpha;
        a.out = (int32_t)out;
        a.in = (int32_t)in;
        a.KT = (int32_t)bd::tiled_k_tiles(in);
        a.units = (int32_t)((in + 127) / 128);   // (in % 128 == 0 but for panels)
        a.wscale = wscale;
        a.inf_in_parts = inf_in_parts ? 1 : 0;
        a.row_blocks = (int32_t)bd::tiled_row_blocks(out);
        a.n_tiles = n;
        const WidePlan p = split & 15     ? WidePlan{split >= kVariantPanels ? bd::kPanelRowBlocks : split >> 4, std::min(split & 15, n), 0.0}
                           : panel_planes ? panel_plan(n, out, in, cus, panel_planes, wscale != nullptr)
                                          : wide_plan(n, t.tokens / launches, out, in, cus, packed_dev != nullptr);
        a.tiles_per_chunk = p.per_chunk;
        for (int i = 0; i < n; ++i) {
            a.tenant[i] = t.tenant[(size_t)(first + i)];
            if (tiled_host) a.signs[i] = tiled_host[a.tenant[i]];
            std::memcpy(a.col_token[i], &t.token[(size_t)(first + i) * 16], 32);
        }
        const hipError_t e = p.R == bd::kPanelRowBlocks ? bd::launch_linear_panel(a, std::max(panel_planes, 1), st) : bd::launch_linear_wide(a, p.R, packed_dev != nullptr, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Where a launch of n tokens (sorted by tenant) is cut into its two column tiles.  Both tiles run as many job slots as the
// one with more jobs needs, so the cut that balances the jobs is taken; of those, one between two tenants (a tenant on both
// sides has its delta streamed twice), then the one nearest the middle.  (18 tokens of 18 tenants as 16 + 2 took nearly as long as 32:
// 274 us for a 7B layer; as 9 + 9 they take 221.)  A column's result does not depend on its tile.
int split_of_launch(const int32_t* tenant_of_token, const int32_t* order, int n, int per_tile, int* jobs = nullptr) {
    int runs_before[2 * bd::kTiledMaxTokens + 1];   // runs_before[i]: tenants among the first i tokens
    runs_before[0] = 0;
    auto new_run = [&](int i) { return i == 0 || tenant_of_token[order[i]] != tenant_of_token[order[i - 1]]; };
    for (int i = 0; i < n; ++i) runs_before[i + 1] = runs_before[i] + (new_run(i) ? 1 : 0);
    int best = per_tile, best_cost = 1 << 30;
    for (int s = n - per_tile; s <= per_tile; ++s) {   // 1 <= n - per_tile <= s: both tiles hold a token
        const int left = runs_before[s], cut = new_run(s) ? 0 : 1, right = runs_before[n] - left + cut;
        const int cost = std::max(left, right) * 1024 + cut * 512 + std::abs(2 * s - n);
        if (cost < best_cost) {
            best_cost = cost;
            best = s;
            if (jobs) *jobs = std::max(left, right);
        }
    }
    return best;
}

// What a batch looks like to the ways of running it: decode launches of 32 tokens of the sorted
// order, which re-read the base per launch but spend nothing on empty rows; the wide kernel and panels, 16-column tiles of one tenant;
// the GEMM, tiles of 32, 64 or 128 rows of one tenant.  A wrong guess costs time, never correctness.
// The estimates for T > 32 were fitted to batches of 33 to 600 tokens of 1 to 64 tenants on 300 .. 12000 x 512 .. 11520 (28672 rows or as long ones are
// extrapolated, here as in the other fits of this file), weights from HBM, replayed from
// graphs (250 row-major, 200 on the serving layout): each is within 10 % at its 10 % and 90 % quantiles (the GEMM's 15 %).  Of 150 other
// batches each, up to 4096 (row-major) or 1500 tokens, 5 % ran more than 8 % (5 %) longer than the quickest of the three ways, 1 % more than 17 % (8 %)
// (before panels).  Up to 32 tokens: few_tokens_wide.
struct BatchShape {
    struct Launch {
        int tokens, tenants, jobs;                       // jobs of its fuller column tile
    };
    int active = 0, tiles16 = 0;
    int64_t tiles32 = 0, tiles64 = 0, tiles128 = 0;      // GEMM tiles by the rows they run
    int64_t runs = 0;                                    // stretches of consecutive tokens of one tenant
    std::vector<Launch> launches;
};
BatchShape batch_shape(const int32_t* tenant_of_token, const std::vector<int32_t>& order) {
    const int64_t T = (int64_t)order.size();
    BatchShape s;
    for (int64_t i = 0; i < T;) {
        int64_t e = i;
        for (; e < T && tenant_of_token[order[(size_t)e]] == tenant_of_token[order[(size_t)i]]; ++e)
            if (e == i || order[(size_t)e] != order[(size_t)e - 1] + 1) ++s.runs;
        const int64_t n = e - i, rest = n % bd::kPrefillTile;
        i = e;
        ++s.active;
        s.tiles16 += (int)((n + 15) / 16);
        s.tiles128 += n / bd::kPrefillTile;
        if (rest > 64) ++s.tiles128;
        else if (rest > 32) ++s.tiles64;
        else if (rest > 0) ++s.tiles32;
    }
    for (int64_t t0 = 0; t0 < T; t0 += kMaxDecodeTokens) {
        const int n = (int)std::min<int64_t>(kMaxDecodeTokens, T - t0);
        const int32_t* const o = order.data() + t0;
        int tenants = 1;
        for (int i = 1; i < n; ++i) tenants += tenant_of_token[o[i]] != tenant_of_token[o[i - 1]] ? 1 : 0;
        int jobs = tenants;
        if (n > bd::kTiledMaxTokens) split_of_launch(tenant_of_token, o, n, bd::kTiledMaxTokens, &jobs);
        s.launches.push_back({n, tenants, jobs});
    }
    return s;
}
// The row-major GEMM.  Per 64-wide k step a tile of 128, 64 or 32 rows takes 1.77, 1.3 or 0.75 us where the compute units are full, plus 2.7 us;
// a last round of at most half of them (whose tiles of 128 rows run as halves) 0.68 us per step.  One tile per compute unit at a time.  The
// token tables come first: from runs (320 to a launch, 0.1 us each) or as they are (960 ints and 2.2 us a launch).
double gemm_us(const BatchShape& s, int64_t out, int64_t in, bool big, int cus) {
    const double steps = (double)in / 64.0;
    const int64_t mtiles = s.tiles32 + s.tiles64 + s.tiles128, runs = s.runs + 3 * mtiles;
    const int64_t by_value = (mtiles * (bd::kPrefillTile + 1) + 959) / 960, by_run = (runs + 319) / 320;
    const double tables = 2.0 + (by_run < by_value ? 0.1 * (double)runs : 2.2 * (double)by_value);
    if (!big) {   // 128 x 128 tiles, two workgroups per compute unit, whatever rows are filled
        const int64_t tiles = mtiles * ((out + 127) / 128);
        return tables + (double)((tiles + 2 * cus - 1) / (2 * cus)) * (steps * 1.9 + 10.0);
    }
    const int64_t tiles = mtiles * ((out + 255) / 256), last = tiles % cus;
    const double full = 2.7 + steps * (s.tiles32 * 0.75 + s.tiles64 * 1.3 + s.tiles128 * 1.77) / (double)mtiles;
    const double rounds = (double)(tiles / cus) * full + (last == 0 ? 0.0 : 2 * last <= cus ? 2.7 + 0.68 * steps : full);
    return tables + std::max(rounds, (double)out * (double)in * (2.0 + (double)s.active / 8.0) / 2.9e6);
}
// The GEMM over the 8-bit base (its tiles as above, 0.62, 1.37 and 1.76 us per step and 7.7 around them) and with k planes (128 x 128 tiles, two workgroups per compute
// unit: 1.2 + 0.4 k us per step while there is one of them per unit, 1.23 + 0.83 k where there are two; a few units with two take 60 % of that way,
// half of them all of it: three planes, 272 workgroups on 256 units 189 us, 222 in panels).  Fitted to 100 prompts of 24 to 4096 tokens of 1 to 16 tenants on
// 500 .. 11008 x 512 .. 11008: 14 % and 9 % at the 10 % and 90 % quantiles.
double gemm_extended_us(const BatchShape& s, int64_t out, int64_t in, bool big, int planes, bool q8, int cus) {
    if (q8 && !big) return gemm_us(s, out, in, false, cus);
    const double steps = (double)in / 64.0;
    const int64_t mtiles = s.tiles32 + s.tiles64 + s.tiles128, runs = s.runs + 3 * mtiles;
    const int64_t by_value = (mtiles * (bd::kPrefillTile + 1) + 959) / 960, by_run = (runs + 319) / 320;
    const double tables = 2.0 + (by_run < by_value ? 0.1 * (double)runs : 2.2 * (double)by_value);
    if (!q8) {
        const double per_unit = (double)(mtiles * ((out + 127) / 128)) / cus, one = 1.2 + 0.4 * planes, two = 1.23 + 0.83 * planes;
        return tables + 3.3 + steps * (per_unit <= 1.0 ? one : per_unit < 1.5 ? one + (two - one) * (0.6 + 0.8 * (per_unit - 1.0)) : std::max(1.0, per_unit / 2.0) * two);
    }
    const int64_t tiles = mtiles * ((out + 255) / 256), last = tiles % cus;
    const double step = (s.tiles32 * 0.62 + s.tiles64 * 1.37 + s.tiles128 * 1.76) / (double)mtiles;
    return tables + (double)(tiles / cus) * (7.7 + steps * step) + (last == 0 ? 0.0 : 7.7 + steps * (2 * last <= cus ? std::min(0.8, step) : step));
}
// k tiles of the wavefronts of a decode launch
double decode_k_tiles(int64_t in, bool rowmajor) {
    const int KT = (int)bd::tiled_k_tiles(in), nw = bd::wide_k_waves(KT);
    int u[8] = {};
    for (int w = 0; w < nw; ++w) u[w] = rowmajor ? (KT - w + nw - 1) / nw : (w + 1) * KT / nw - w * KT / nw;
    return steps_of_waves(u);
}
// Decode launches over `row_blocks` (those of a group together, `elems` their weights): about 6 us each, and the longer of the
// tasks (per row block, k tile and column tile 1.7 us and 0.2 (row-major) or 0.13 per job slot, slots in twos) and the
// bytes at 2.9 or 3.3 TB/s (32 tokens of 8 tenants on 4096 x 4096: 19 us).  The vector-ALU kernel streams everything at 1.3 TB/s plus 8 us.
double decode_us(const BatchShape& s, int64_t row_blocks, double elems, int64_t in, int cus, bool tiled, bool on_matrix_cores) {
    double us = 0.0;
    const double tasks = (double)((row_blocks + cus - 1) / cus) * decode_k_tiles(in, !tiled);
    for (const auto& l : s.launches) {
        const double bytes = elems * (2.0 + (double)l.tenants / 8.0), slots = (double)((l.jobs + 1) / 2 * 2), ct = l.tokens > 16 ? 2.0 : 1.0;
        if (!on_matrix_cores) us += 8.0 + bytes / 1.3e6;
        else if (tiled) us += 6.2 + std::max(tasks * ct * (1.8 + 0.135 * slots), bytes / 3.3e6);
        else us += 6.1 + std::max(tasks * ct * (1.65 + 0.21 * slots), bytes / 2.9e6);
    }
    return us;
}
// Row-major batches that fit one decode launch.  That launch takes every job slot through every fetch and waits for memory once per task; the
// wide and panel kernels pad each tenant to 16 columns but share what they fetch between them (us, decode / the other): 4501 x 512 31 tokens of 2
// tenants 14.6 / 7.3, 994 x 640 29 of 17 15.6 / 7.2, 953 x 4736 24 of 6 19.3 / 13.5, 11578 x 9216 21 of 2 73 / 54; 11708 x 4224 9 of 9 49 / 77,
// 5827 x 2304 9 of 8 18 / 22, 3173 x 10624 2 of 2 22 / 28.  Both estimates are fitted to 500 batches of 1 to 32 tokens on 300 .. 12000 x 512 .. 11520
// (decode 15 %, the others 8 % at the 10 % and 90 % quantiles) apart from those above, which are for several launches or many column tiles.
bool few_tokens_wide(const BatchShape& s, int64_t out, int64_t in, int cus) {
    const double elems = (double)out * (double)in, bytes = elems * (2.0 + (double)s.active / 8.0), units = wide_units(in, true);
    const auto& l = s.launches[0];
    const double tasks = (double)((bd::tiled_row_blocks(out) + cus - 1) / cus) * decode_k_tiles(in, true) * (l.tokens > 16 ? 2.0 : 1.0);
    const double by_decode = 5.35 + std::max(tasks * (1.73 + 0.273 * (double)((l.jobs + 1) / 2 * 2)), bytes / 4.0e6);
    const double limit = 0.86 * by_decode;   // at 0.88 none of 1000 is slower by more than 2.6 %, at 1.0 19 of 500 are by 3 to 15 %
    const double least = 5.7 + bytes / 3.96e6;
    if (limit <= std::max(least, 4.8 + 1.31 * units)) return false;   // no plan is quicker: the smallest calls need no search
    const int n = s.tiles16;
    const WidePlan p = wide_plan(n, l.tokens, out, in, cus, true);
    const int64_t groups = (bd::tiled_row_blocks(out) + p.R - 1) / p.R, chunks = (n + p.per_chunk - 1) / p.per_chunk, per_xcd = std::max(1, cus / 8);
    const double rounds = (double)(((groups + 7) / 8 * chunks + per_xcd - 1) / per_xcd);
    double us = 1.5;
    if (p.R == bd::kPanelRowBlocks)
        us += rounds * (4.0 + 0.367 * (double)(((in + 127) / 128 + 1) / 2 * std::max(2, p.per_chunk))) + (double)chunks * elems * 0.064e-6;
    else if (p.R == 2)
        us += rounds * (4.2 + 0.783 * units * (double)((p.per_chunk + 1) / 2 * 2)) + (double)chunks * elems * 0.15e-6;
    else
        us += rounds * (3.3 + 1.31 * units) + (double)chunks * elems * 0.166e-6;
    return std::max(us, least) < limit;
}
// The same question on the serving layout, for one matrix and one plane (the same bits either way); a decode launch streams it better, so the line
// lies further out: 414 x 5376 31 tokens of 14 tenants 23.8 / 12.4, 14008 x 512 28 of 2 22.3 / 11.4, 15357 x 1280 31 of 1 27.5 / 16.7, 1081 x 3584 32 of 4
// 16.1 / 10.8; 8681 x 768 7 of 7 15.0 / 18.7, 4430 x 4608 19 of 4 24.0 / 25.9, 452 x 3072 1 token 7.2 / 8.4.  Fitted to 400 batches (decode 15 %, wide 9 %).
bool few_tokens_wide_tiled(const BatchShape& s, int64_t out, int64_t in, int cus) {
    const double elems = (double)out * (double)in, bytes = elems * (2.0 + (double)s.active / 8.0), units = wide_units(in, false);
    const auto& l = s.launches[0];
    const double tasks = (double)((bd::tiled_row_blocks(out) + cus - 1) / cus) * decode_k_tiles(in, false) * (l.tokens > 16 ? 2.0 : 1.0);
    const double by_decode = 4.69 + std::max(tasks * (1.714 + 0.191 * (double)((l.jobs + 1) / 2 * 2)), bytes / 5.39e6);
    const double limit = 0.82 * by_decode;   // of the 400 none is then slower; at 0.9 3 are by 3 to 14 %, at 1.0 13
    const double least = 6.0 + bytes / 3.6e6;
    if (limit <= std::max(least, 4.55 + 1.12 * units)) return false;   // no plan is quicker: the smallest calls need no search
    const int n = s.tiles16, KT = (int)bd::tiled_k_tiles(in);
    const WidePlan p = wide_plan(n, l.tokens, out, in, cus, false);
    const int64_t per_group = p.R * (8 / bd::wide_k_waves(KT)), groups = (bd::tiled_row_blocks(out) + per_group - 1) / per_group;
    const int64_t chunks = (n + p.per_chunk - 1) / p.per_chunk, per_xcd = std::max(1, cus / 8);
    const double rounds = (double)(((groups + 7) / 8 * chunks + per_xcd - 1) / per_xcd), run = (double)((p.per_chunk + 1) / 2 * 2);
    const double us = p.R == 2 ? rounds * (5.03 + 0.701 * units * run) + (double)chunks * elems * 0.047e-6
                               : rounds * (2.25 + 0.56 * units * run) + (double)chunks * elems * 0.136e-6;
    return std::max(2.3 + us, least) < limit;
}

}  // namespace

extern "C" {

const char* bd_status_string(bd_status s) {
    switch (s) {
        case BD_OK: return "ok";
        case BD_ERR_NULL: return "a required pointer is NULL";
        case BD_ERR_SHAPE: return "bad shape: negative, too large, or in not a multiple of 32";
        case BD_ERR_ALIGN: return "a tensor pointer is not 16-byte aligned";
        case BD_ERR_TENANT: return "tenant id outside [0, n_tenants)";
        case BD_ERR_WORKSPACE: return "workspace missing, too small or misaligned";
        case BD_ERR_DEVICE: return "the HIP runtime reported an error";
        case BD_ERR_UNSUPPORTED: return "unsupported op or kernel variant for these sizes";
        case BD_ERR_ALIAS: return "the output overlaps an input";
        case BD_ERR_FORMAT: return "malformed delta image";
        case BD_ERR_IO: return "file could not be opened, read or written";
        case BD_ERR_TOO_LARGE: return "size beyond the fixed limit of this entry point";
    }
    return "unknown status";
}

int bd_version(void) { return kVersion; }

size_t bd_workspace_bytes(bd_op op, int64_t T, int64_t out, int64_t in, int32_t n_tenants) {
    if (out < 0 || in < 0 || in % 32 != 0) return 0;
    switch (op) {
        case BD_OP_COMPRESS: return (size_t)bd::kCompressMaxBlocks * sizeof(double);
        case BD_OP_PACK_SIGNS: return 0;
        case BD_OP_LINEAR_MULTITENANT: return prefill_workspace_bytes(T, n_tenants);
        case BD_OP_LINEAR_GEMM: return prefill_table_bytes(T, n_tenants);
        case BD_OP_LINEAR_TILED_GEMM: return tiled_gemm_workspace_bytes(T, n_tenants);
    }
    return 0;
}

bd_status bd_pack_signs(const uint16_t* delta_f16, int64_t out, int64_t in, uint32_t* packed, void* stream) {
    if (out < 0 || in < 0 || in % 32 != 0) return BD_ERR_SHAPE;
    if (out == 0 || in == 0) return BD_OK;
    if (!delta_f16 || !packed) return BD_ERR_NULL;
    if (misaligned(delta_f16, 16) || misaligned(packed, 16)) return BD_ERR_ALIGN;
    if (overlaps(packed, (size_t)out * in / 8, delta_f16, (size_t)out * in * 2)) return BD_ERR_ALIAS;
    return bd::launch_pack_signs(delta_f16, out, in, packed, (hipStream_t)stream) == hipSuccess ? BD_OK : BD_ERR_DEVICE;
}

bd_status bd_compress(const uint16_t* w_base_f16, const uint16_t* w_ft_f16, int64_t out, int64_t in, uint32_t* packed,
                      float* alpha, void* workspace, size_t workspace_bytes, void* stream) {
    if (out < 0 || in < 0 || in % 32 != 0) return BD_ERR_SHAPE;
    if (!alpha) return BD_ERR_NULL;
    if (misaligned(alpha, 4)) return BD_ERR_ALIGN;
    const bool empty = (out == 0 || in == 0);
    if (!empty) {
        if (!w_base_f16 || !w_ft_f16 || !packed) return BD_ERR_NULL;
        if (misaligned(w_base_f16, 16) || misaligned(w_ft_f16, 16) || misaligned(packed, 16)) return BD_ERR_ALIGN;
        const size_t wbytes = (size_t)out * in * 2, pbytes = (size_t)out * in / 8;
        if (overlaps(packed, pbytes, w_base_f16, wbytes) || overlaps(packed, pbytes, w_ft_f16, wbytes)) return BD_ERR_ALIAS;
    }
    const size_t need = bd_workspace_bytes(BD_OP_COMPRESS, 0, out, in, 1);
    if (!workspace || workspace_bytes < need || misaligned(workspace, 256)) return BD_ERR_WORKSPACE;
    return bd::launch_compress(w_base_f16, w_ft_f16, out, in, packed, alpha, (double*)workspace,
                               (hipStream_t)stream) == hipSuccess
               ? BD_OK
               : BD_ERR_DEVICE;
}

bd_status bd_compress_noalloc(const uint16_t* w_base_f16, const uint16_t* w_ft_f16, int64_t out, int64_t in,
                              uint32_t* packed, float* alpha, void* stream) {
    if (out < 0 || in < 0 || in % 32 != 0) return BD_ERR_SHAPE;
    if (!alpha) return BD_ERR_NULL;
    if (misaligned(alpha, 4)) return BD_ERR_ALIGN;
    // the size limit of this entry point, checked without overflow (out, in >= 0 here)
    if (out > 0 && in > BD_COMPRESS_NOALLOC_MAX_ELEMENTS / out) return BD_ERR_TOO_LARGE;
    if (out > 0 && in > 0) {
        if (!w_base_f16 || !w_ft_f16 || !packed) return BD_ERR_NULL;
        if (misaligned(w_base_f16, 16) || misaligned(w_ft_f16, 16) || misaligned(packed, 16)) return BD_ERR_ALIGN;
        const size_t wbytes = (size_t)out * in * 2, pbytes = (size_t)out * in / 8;
        if (overlaps(packed, pbytes, w_base_f16, wbytes) || overlaps(packed, pbytes, w_ft_f16, wbytes)) return BD_ERR_ALIAS;
    }
    return bd::launch_compress_noalloc(w_base_f16, w_ft_f16, out, in, packed, alpha, (hipStream_t)stream) == hipSuccess
               ? BD_OK
               : BD_ERR_DEVICE;
}

bd_status bd_compress_batch(int32_t n, const uint16_t* const* w_base_f16, const uint16_t* const* w_ft_f16,
                            const int64_t* out, const int64_t* in, uint32_t* const* packed, float* alpha, void* workspace,
                            size_t workspace_bytes, void* stream) {
    if (n < 0) return BD_ERR_SHAPE;
    if (n == 0) return BD_OK;
    if (!w_base_f16 || !w_ft_f16 || !out || !in || !packed || !alpha) return BD_ERR_NULL;
    if (misaligned(alpha, 4)) return BD_ERR_ALIGN;
    for (int32_t m = 0; m < n; ++m) {
        if (out[m] < 0 || in[m] < 0 || in[m] % 32 != 0) return BD_ERR_SHAPE;
        if (out[m] == 0 || in[m] == 0) continue;
        if (!w_base_f16[m] || !w_ft_f16[m] || !packed[m]) return BD_ERR_NULL;
        if (misaligned(w_base_f16[m], 16) || misaligned(w_ft_f16[m], 16) || misaligned(packed[m], 16)) return BD_ERR_ALIGN;
        const size_t wbytes = (size_t)out[m] * in[m] * 2, pbytes = (size_t)out[m] * in[m] / 8;
        for (int32_t o = 0; o < n; ++o) {   // no plane of signs may lie over any matrix that is still to be read
            if (out[o] == 0 || in[o] == 0) continue;
            const size_t obytes = (size_t)out[o] * in[o] * 2;
            if (overlaps(packed[m], pbytes, w_base_f16[o], obytes) || overlaps(packed[m], pbytes, w_ft_f16[o], obytes))
                return BD_ERR_ALIAS;
            if (o != m && overlaps(packed[m], pbytes, packed[o], (size_t)out[o] * in[o] / 8)) return BD_ERR_ALIAS;
        }
        (void)wbytes;
    }
    const size_t need = (size_t)BD_COMPRESS_BATCH_MAX * bd_workspace_bytes(BD_OP_COMPRESS, 0, 1, 32, 1);
    if (!workspace || workspace_bytes < need || misaligned(workspace, 256)) return BD_ERR_WORKSPACE;
    for (int32_t m0 = 0; m0 < n; m0 += bd::kCompressBatchMax) {   // launches of up to 8 matrices, in stream order
        bd::CompressBatch a;
        std::memset(&a, 0, sizeof(a));
        a.n = std::min<int32_t>(bd::kCompressBatchMax, n - m0);
        for (int i = 0; i < a.n; ++i) {
            const int32_t m = m0 + i;
            a.base[i] = w_base_f16[m];
            a.ft[i] = w_ft_f16[m];
            a.packed[i] = packed[m];
            a.n_vec[i] = out[m] * in[m] / 8;
        }
        if (bd::launch_compress_batch(a, alpha + m0, (double*)workspace, (hipStream_t)stream) != hipSuccess) return BD_ERR_DEVICE;
    }
    return BD_OK;
}

bd_status bd_compress_iterated(const uint16_t* w_base_f16, const uint16_t* w_ft_f16, int64_t out, int64_t in, int32_t k,
                               uint32_t* packed, float* alpha, void* workspace, size_t workspace_bytes, void* stream) {
    if (out < 0 || in < 0 || in % 32 != 0 || k < 1 || k > bd::kCompressMaxPlanes) return BD_ERR_SHAPE;
    if (!alpha) return BD_ERR_NULL;
    if (misaligned(alpha, 4)) return BD_ERR_ALIGN;
    const bool empty = (out == 0 || in == 0);
    const size_t plane_words = (size_t)out * in / 32;
    if (!empty) {
        if (!w_base_f16 || !w_ft_f16 || !packed) return BD_ERR_NULL;
        if (misaligned(w_base_f16, 16) || misaligned(w_ft_f16, 16) || misaligned(packed, 16)) return BD_ERR_ALIGN;
        const size_t wbytes = (size_t)out * in * 2, pbytes = plane_words * 4 * (size_t)k;
        if (overlaps(packed, pbytes, w_base_f16, wbytes) || overlaps(packed, pbytes, w_ft_f16, wbytes)) return BD_ERR_ALIAS;
    }
    const size_t need = bd_workspace_bytes(BD_OP_COMPRESS, 0, out, in, 1);
    if (!workspace || workspace_bytes < need || misaligned(workspace, 256)) return BD_ERR_WORKSPACE;
    // iteration j reads the scales 0 .. j-1 that the iterations before it left in `alpha` (same stream)
    for (int j = 0; j < k; ++j)
        if (bd::launch_compress(w_base_f16, w_ft_f16, out, in, packed + (size_t)j * plane_words, alpha + j, (double*)workspace,
                                (hipStream_t)stream, alpha, j) != hipSuccess)
            return BD_ERR_DEVICE;
    return BD_OK;
}

namespace {
bd_status tiled_linear_impl(int32_t n_mats, const uint16_t* x_f16, const uint16_t* const* w_tiled,
                            const uint32_t* const* tiled_by_mat_tenant, const float* const* alpha_by_mat,
                            const int32_t* tenant_of_token, uint16_t* const* y_f16, int64_t T, const int64_t* out,
                            int64_t in, int32_t n_tenants, int32_t k, void* stream, bool q8,
                            const uint32_t* const* packed_rowmajor_dev, const float* wscale_rowmajor = nullptr, int32_t variant = 0);
}

bd_status bd_linear_multitenant_variant(const uint16_t* x_f16, const uint16_t* w_base_f16,
                                        const uint32_t* const* packed_by_tenant, const float* alpha_by_tenant,
                                        const int32_t* tenant_of_token, uint16_t* y_f16, int64_t T, int64_t out,
                                        int64_t in, int32_t n_tenants, void* workspace, size_t workspace_bytes,
                                        void* stream, int32_t variant) {
    const bd_status st = check_linear_args(x_f16, w_base_f16, packed_by_tenant, alpha_by_tenant, tenant_of_token, y_f16,
                                           T, out, in, n_tenants);
    if (st != BD_OK) return st;
    const bool merged_variant = variant == kVariantPrefillMerged;
    const bool big_variant = variant == kVariantPrefillBig || variant == kVariantPrefillBig8 || variant == kVariantPrefillBigWhole ||
                             merged_variant;
    const bool prefill_variant = variant == kVariantPrefillSmall || big_variant;
    const int wide_split = wide_split_of_variant(variant, in, true);
    if (variant != 0 && variant != kVariantRowWave && variant != kVariantRowMajorMfma && !prefill_variant && wide_split < 0)
        return BD_ERR_UNSUPPORTED;
    if (T == 0 || out == 0) return BD_OK;
    std::vector<int32_t> order;
    auto wide = [&](const int split) {
        return run_wide(wide_tiles(tenant_of_token, order), x_f16, w_base_f16, packed_by_tenant, nullptr, alpha_by_tenant, y_f16, out, in,
                        (hipStream_t)stream, split, split >= kVariantPanels ? 1 : 0) == hipSuccess
                   ? BD_OK
                   : BD_ERR_DEVICE;
    };
    if (wide_split >= 0 && !wide_fits(T, out, in)) return BD_ERR_UNSUPPORTED;
    if (T > kMaxDecodeTokens || wide_split >= 0) order = order_by_tenant(tenant_of_token, T, n_tenants);
    if (wide_split >= 0) return wide(wide_split);
    // 128-bit sign loads need whole, aligned 4-word groups; 32-bit lane offsets need tensors below 4 GiB
    const bool mfma_ok = (in % 128 == 0) && in > 0 && (uint64_t)out * (uint64_t)in * 2 < ((uint64_t)1 << 32) &&
                         (uint64_t)T * (uint64_t)in * 2 < ((uint64_t)1 << 32);
    if (variant >= 2 && !prefill_variant && !mfma_ok) return BD_ERR_UNSUPPORTED;
    if (variant == 0 && T <= kMaxDecodeTokens && mfma_ok && wide_fits(T, out, in)) {
        order = order_by_tenant(tenant_of_token, T, n_tenants);
        if (few_tokens_wide(batch_shape(tenant_of_token, order), out, in, cus_or_256())) return wide(0);
    }
    int use = variant;
    if (use == 0) use = mfma_ok ? kVariantRowMajorMfma : kVariantRowWave;

    hipStream_t hs = (hipStream_t)stream;
    // More than one decode launch worth of tokens: the prefill GEMM, if the caller brought its workspace
    // (without one the call still works, as a sequence of decode launches that re-read the base).
    const size_t need = prefill_workspace_bytes(T, n_tenants);
    const bool can_prefill = need > 0 && in > 0 && workspace && workspace_bytes >= need && !misaligned(workspace, 256);
    if (prefill_variant && !can_prefill) return need > 0 && in > 0 ? BD_ERR_WORKSPACE : BD_ERR_UNSUPPORTED;
    if (big_variant && !bd::prefill_big_fits(T, out, in)) return BD_ERR_UNSUPPORTED;
    const bool big_default = out >= 256 && bd::prefill_big_fits(T, out, in);
    bool gemm_pays = prefill_variant;
    if (variant == 0 && T > kMaxDecodeTokens && in > 0) {   // the library's choice, by estimated time
        const BatchShape shape = batch_shape(tenant_of_token, order);
        const int cus = cus_or_256();
        const double by_decode = decode_us(shape, bd::tiled_row_blocks(out), (double)out * (double)in, in, cus, false, mfma_ok);
        const double by_gemm = can_prefill ? gemm_us(shape, out, in, big_default, cus) : 1e30;
        // Halves of five units: a panel fetches and turns the signs of four units at a time, here three for nothing, and its estimate is a tenth short.
        // Decode launches / panels: 5250 x 1280 64 tokens of 58 tenants 60 / 71, 10080 x 1152 58 of 44 73 / 80, 5131 x 1152 73 of 66 76 / 82 (11 of 22
        // such batches between 3 and 15 %); beyond that line 5870 x 1152 41 of 36 45.5 / 42.7, 3051 x 1152 46 of 41 30.9 / 29.0.
        const double against_decode = (in / 128 + 1) / 2 == 5 ? 0.9 : 1.0;
        if (mfma_ok && wide_fits(T, out, in) &&
            wide_us(shape.tiles16, T, shape.active, out, in, cus, true) < std::min(against_decode * by_decode, by_gemm))
            return wide(0);
        gemm_pays = by_gemm < by_decode;
    }
    if (can_prefill && gemm_pays) {
        // the large tile (one workgroup per CU, 256 output features wide) pays off when there are at least that many
        int big_waves = 0;
        if (variant == kVariantPrefillBig8) big_waves = 8;
        if (variant == kVariantPrefillBig || variant == kVariantPrefillBigWhole || variant == kVariantPrefillMerged ||
            (variant == 0 && big_default))
            big_waves = 4;
        return run_prefill(x_f16, w_base_f16, packed_by_tenant, alpha_by_tenant, tenant_of_token, order, y_f16, T, out, in,
                           workspace, hs, big_waves, variant != kVariantPrefillBigWhole, 0, nullptr, merged_variant) == hipSuccess
                   ? BD_OK
                   : BD_ERR_DEVICE;
    }
    if (prefill_variant) use = mfma_ok ? kVariantRowMajorMfma : kVariantRowWave;   // not reached: can_prefill held above
    if (use == kVariantRowMajorMfma && in > 0)
        // the decode kernel of the serving path, reading the row-major tensors as they are; all tokens are grouped by
        // tenant first, then cut into launches of 32
        return tiled_linear_impl(1, x_f16, &w_base_f16, nullptr, &alpha_by_tenant, tenant_of_token, &y_f16, T, &out, in,
                                 n_tenants, 1, stream, false, packed_by_tenant);
    for (int64_t t0 = 0; t0 < T; t0 += kMaxDecodeTokens) {
        const int n = (int)std::min<int64_t>(kMaxDecodeTokens, T - t0);
        DecodeMeta meta;
        build_meta(tenant_of_token, t0, n, &meta);
        const uint16_t* xs = x_f16 + t0 * in;
        uint16_t* ys = y_f16 + t0 * out;
        hipError_t e;
        // the vector-ALU kernel; also the empty reduction, y = 0 (its loop body never runs)
        e = bd::launch_linear_rowwave(xs, w_base_f16, packed_by_tenant, alpha_by_tenant, meta, ys, out, in, hs);
        if (e != hipSuccess) return BD_ERR_DEVICE;
    }
    return BD_OK;
}

bd_status bd_linear_multitenant(const uint16_t* x_f16, const uint16_t* w_base_f16,
                                const uint32_t* const* packed_by_tenant, const float* alpha_by_tenant,
                                const int32_t* tenant_of_token, uint16_t* y_f16, int64_t T, int64_t out, int64_t in,
                                int32_t n_tenants, void* workspace, size_t workspace_bytes, void* stream) {
    return bd_linear_multitenant_variant(x_f16, w_base_f16, packed_by_tenant, alpha_by_tenant, tenant_of_token, y_f16, T,
                                         out, in, n_tenants, workspace, workspace_bytes, stream, 0);
}

// ---- tiled serving layout ------------------------------------------------------------------

namespace {

bool tiled_shape_ok(int64_t out, int64_t in) {
    if (out < 0 || in < 0 || in % 32 != 0) return false;
    if (out > ((int64_t)1 << 31) - 16 || in > ((int64_t)1 << 31) - 256) return false;
    // 32-bit byte offsets inside one tiled tensor
    const uint64_t tiles = (uint64_t)bd::tiled_row_blocks(out) * (uint64_t)bd::tiled_k_tiles(in);
    return tiles * (uint64_t)bd::kTileBaseBytes < ((uint64_t)1 << 32);
}

}  // namespace

size_t bd_tiled_base_bytes(int64_t out, int64_t in) {
    if (!tiled_shape_ok(out, in)) return 0;
    return (size_t)(bd::tiled_row_blocks(out) * bd::tiled_k_tiles(in)) * bd::kTileBaseBytes;
}

size_t bd_tiled_signs_bytes(int64_t out, int64_t in) {
    if (!tiled_shape_ok(out, in)) return 0;
    return (size_t)(bd::tiled_row_blocks(out) * bd::tiled_k_tiles(in)) * bd::kTileSignBytes;
}

bd_status bd_tile_base(const uint16_t* w_f16, int64_t out, int64_t in, uint16_t* w_tiled, void* stream) {
    if (!tiled_shape_ok(out, in)) return BD_ERR_SHAPE;
    if (out == 0 || in == 0) return BD_OK;
    if (!w_f16 || !w_tiled) return BD_ERR_NULL;
    if (misaligned(w_f16, 16) || misaligned(w_tiled, 16)) return BD_ERR_ALIGN;
    if (overlaps(w_tiled, bd_tiled_base_bytes(out, in), w_f16, (size_t)out * in * 2)) return BD_ERR_ALIAS;
    return bd::launch_tile_base(w_f16, out, in, w_tiled, (hipStream_t)stream) == hipSuccess ? BD_OK : BD_ERR_DEVICE;
}

bd_status bd_tile_signs(const uint32_t* packed, int64_t out, int64_t in, uint32_t* signs_tiled, void* stream) {
    if (!tiled_shape_ok(out, in)) return BD_ERR_SHAPE;
    if (out == 0 || in == 0) return BD_OK;
    if (!packed || !signs_tiled) return BD_ERR_NULL;
    if (misaligned(packed, 16) || misaligned(signs_tiled, 16)) return BD_ERR_ALIGN;
    if (overlaps(signs_tiled, bd_tiled_signs_bytes(out, in), packed, (size_t)out * in / 8)) return BD_ERR_ALIAS;
    return bd::launch_tile_signs(packed, out, in, signs_tiled, (hipStream_t)stream) == hipSuccess ? BD_OK : BD_ERR_DEVICE;
}

namespace {

// The tiled linear over n_mats matrices that share x, with k sign planes per tenant (k = 1: plain 1-bit
// deltas).  Pointer table index: (m * n_tenants + tenant) * k + plane; scale index: tenant * k + plane.
// q8: w_tiled point at 8-bit base tiles followed by their per-row scales (bd_tile_base_q8).
// packed_rowmajor_dev != NULL: the row-major entry point.  w_tiled[0] is then W [out, in] row-major, the deltas are
// reached through that DEVICE table of n_tenants pointers (tiled_by_mat_tenant is not used), n_mats = k = 1.
bd_status tiled_linear_impl(int32_t n_mats, const uint16_t* x_f16, const uint16_t* const* w_tiled,
                            const uint32_t* const* tiled_by_mat_tenant, const float* const* alpha_by_mat,
                            const int32_t* tenant_of_token, uint16_t* const* y_f16, int64_t T, const int64_t* out,
                            int64_t in, int32_t n_tenants, int32_t k, void* stream, bool q8,
                            const uint32_t* const* packed_rowmajor_dev, const float* wscale_rowmajor, int32_t variant) {
    const bool rm = packed_rowmajor_dev != nullptr;
    if (rm && (n_mats != 1 || in % 128 != 0 || (q8 && (!wscale_rowmajor || k != 1)))) return BD_ERR_UNSUPPORTED;
    if (n_mats < 1 || n_mats > bd::kTiledMaxMats) return BD_ERR_SHAPE;
    if (k < 1 || k > bd::kTiledMaxPlanes) return BD_ERR_SHAPE;
    if (!out) return BD_ERR_NULL;
    if (T < 0 || n_tenants < 0 || T > 65535) return BD_ERR_SHAPE;
    int64_t row_blocks = 0;
    for (int m = 0; m < n_mats; ++m) {
        if (!tiled_shape_ok(out[m], in)) return BD_ERR_SHAPE;
        row_blocks += bd::tiled_row_blocks(out[m]);
    }
    if (row_blocks > 0x7fffffff) return BD_ERR_SHAPE;
    if ((uint64_t)T * (uint64_t)in * 2 >= ((uint64_t)1 << 32)) return BD_ERR_SHAPE;   // 32-bit byte offsets into x
    if (T == 0 || row_blocks == 0) return BD_OK;
    if (in == 0) {   // empty reduction: y = 0, nothing else is read
        if (!y_f16) return BD_ERR_NULL;
        for (int m = 0; m < n_mats; ++m)
            if (out[m] > 0 && !y_f16[m]) return BD_ERR_NULL;
        for (int m = 0; m < n_mats; ++m)
            if (out[m] > 0 && bd::launch_fill_zero_u16(y_f16[m], T * out[m], (hipStream_t)stream) != hipSuccess) return BD_ERR_DEVICE;
        return BD_OK;
    }
    if (!x_f16 || !w_tiled || (!rm && !tiled_by_mat_tenant) || !alpha_by_mat || !tenant_of_token || !y_f16) return BD_ERR_NULL;
    if (misaligned(x_f16, 16)) return BD_ERR_ALIGN;
    for (int64_t t = 0; t < T; ++t)
        if (tenant_of_token[t] < 0 || tenant_of_token[t] >= n_tenants) return BD_ERR_TENANT;
    for (int m = 0; m < n_mats; ++m) {
        if (out[m] == 0) continue;
        if (!w_tiled[m] || !alpha_by_mat[m] || !y_f16[m]) return BD_ERR_NULL;
        if (misaligned(w_tiled[m], 16) || misaligned(y_f16[m], 2) || misaligned(alpha_by_mat[m], 4)) return BD_ERR_ALIGN;
        const size_t ybytes = (size_t)T * out[m] * 2;
        const size_t wbytes = rm ? (size_t)out[m] * in * (q8 ? 1 : 2) : (q8 ? bd_tiled_base_q8_bytes(out[m], in) : bd_tiled_base_bytes(out[m], in));
        if (overlaps(y_f16[m], ybytes, x_f16, (size_t)T * in * 2) || overlaps(y_f16[m], ybytes, w_tiled[m], wbytes))
            return BD_ERR_ALIAS;
        for (int64_t t = 0; t < T && !rm; ++t)
            for (int j = 0; j < k; ++j) {
                const uint32_t* p = tiled_by_mat_tenant[((size_t)m * n_tenants + tenant_of_token[t]) * k + j];
                if (!p) return BD_ERR_NULL;
                if (misaligned(p, 16)) return BD_ERR_ALIGN;
            }
    }
    const std::vector<int32_t> order = order_by_tenant(tenant_of_token, T, n_tenants);
    // Serving layout, one plane: the wide kernel, a launch per matrix, where its estimate is below that of the decode launches, which take
    // the matrices of a group together (so a group of a single launch's tokens stays with them).
    const int wide_split = wide_split_of_variant(variant, in, false);
    const bool few = T <= bd::kMaxDecodeTokens;
    if (wide_split >= 0 || (!rm && !q8 && k == 1 && variant == 0 && (!few || n_mats == 1))) {
        bool fits = true;
        for (int m = 0; m < n_mats; ++m) fits = fits && (out[m] == 0 || wide_fits(T, out[m], in));
        if (wide_split >= 0 && !fits) return BD_ERR_UNSUPPORTED;
        bool wide = wide_split >= 0;
        if (!wide && fits) {
            const BatchShape shape = batch_shape(tenant_of_token, order);
            const int cus = cus_or_256();
            double us = 0.0, elems = 0.0;
            for (int m = 0; m < n_mats && !few; ++m) {
                if (out[m] == 0) continue;
                us += wide_us(shape.tiles16, T, shape.active, out[m], in, cus, false);
                elems += (double)out[m] * (double)in;
            }
            wide = few ? few_tokens_wide_tiled(shape, out[0], in, cus) : us < decode_us(shape, row_blocks, elems, in, cus, true, true);
        }
        if (wide) {
            const WideTiles tiles = wide_tiles(tenant_of_token, order);
            for (int m = 0; m < n_mats; ++m)
                if (out[m] > 0 && run_wide(tiles, x_f16, w_tiled[m], nullptr, tiled_by_mat_tenant + (size_t)m * n_tenants, alpha_by_mat[m],
                                           y_f16[m], out[m], in, (hipStream_t)stream, std::max(wide_split, 0), 0, nullptr,
                                           few && wide_split < 0) != hipSuccess)   // (a group of that size is a decode launch)
                    return BD_ERR_DEVICE;
            return BD_OK;
        }
    }
    // A token takes k columns (one per plane) of a 16-column tile; a launch covers two tiles.  More tokens than one
    // launch takes: all of them are sorted by tenant first (stable), so that a tenant's tokens share launches and
    // its delta is streamed as few times as possible; the kernel finds the rows of x and y through the token ids.
    const int per_tile = bd::kTiledMaxTokens / k;
    const int per_launch = per_tile * bd::kTiledMaxCt;
    for (int64_t t0 = 0; t0 < T; t0 += per_launch) {
        const int n = (int)std::min<int64_t>(per_launch, T - t0);
        bd::TiledArgs a;
        std::memset(&a, 0, sizeof(a));
        a.x = x_f16;
        a.in = (int32_t)in;
        a.KT = (int32_t)bd::tiled_k_tiles(in);
        a.n_ct = n > per_tile ? 2 : 1;
        a.planes = k;
        a.packed_by_tenant = packed_rowmajor_dev;
        int32_t rb = 0;
        int mats = 0;
        int mat_of[bd::kTiledMaxMats] = {0, 0, 0};
        for (int m = 0; m < n_mats; ++m) {
            if (out[m] == 0) continue;
            a.wt[mats] = w_tiled[m];
            a.y[mats] = y_f16[m];
            a.alpha[mats] = alpha_by_mat[m];
            if (q8 && rm)
                a.wscale[mats] = wscale_rowmajor;
            else if (q8)   // the scales follow the tiles
                a.wscale[mats] = (const float*)((const unsigned char*)w_tiled[m] +
                                                (size_t)(bd::tiled_row_blocks(out[m]) * bd::tiled_k_tiles(in)) * bd::kTileBaseQ8Bytes);
            a.out[mats] = (int32_t)out[m];
            rb += (int32_t)bd::tiled_row_blocks(out[m]);
            a.rb_end[mats] = rb;
            mat_of[mats] = m;
            ++mats;
        }
        a.n_mats = mats;
        int max_jobs = 1;
        const int first_tile = a.n_ct == 2 ? split_of_launch(tenant_of_token, order.data() + t0, n, per_tile) : n;
        for (int ct = 0; ct < bd::kTiledMaxCt; ++ct) {
            // a column tile beyond n_ct mirrors tile 0 (never read by the kernel, but every pointer stays valid)
            const int src = ct < a.n_ct ? ct : 0;
            const int tok_begin = src * first_tile, tok_end = src == 0 ? first_tile : n;
            int n_runs = 0, run_tenant[bd::kTiledMaxTokens];
            int col = 0;
            for (int i = tok_begin; i < tok_end; ++i) {
                const int tok = order[(size_t)(t0 + i)];
                const int tenant = tenant_of_token[tok];
                if (n_runs == 0 || run_tenant[n_runs - 1] != tenant) run_tenant[n_runs++] = tenant;
                for (int j = 0; j < k; ++j, ++col) {   // the token's columns: plane j is job slot (run, j)
                    a.col_token[ct][col] = tok;
                    a.col_tenant[ct][col] = tenant * k + j;
                    a.col_job[ct][col] = (n_runs - 1) * k + j;
                    a.col_span[ct][col] = j == 0 ? k : 0;
                }
            }
            a.T[ct] = col;
            for (; col < bd::kTiledMaxTokens; ++col) a.col_job[ct][col] = -1;
            const int n_jobs = n_runs * k;
            max_jobs = std::max(max_jobs, n_jobs);
            for (int sl = 0; sl < bd::kTiledMaxJobs; ++sl) {   // slots beyond the jobs repeat slot 0 (never selected)
                const int s = sl < n_jobs ? sl : 0;
                a.job_tenant[ct][sl] = run_tenant[s / k] * k + s % k;   // index into the caller's table: (tenant, plane)
                for (int mi = 0; mi < mats && !rm; ++mi)
                    a.signs[ct][mi][sl] = tiled_by_mat_tenant[((size_t)mat_of[mi] * n_tenants + run_tenant[s / k]) * k + s % k];
            }
        }
        const hipError_t e = rm   ? (q8 ? bd::launch_linear_decode_rowmajor_q8(a, max_jobs, (hipStream_t)stream)
                                        : bd::launch_linear_decode_rowmajor(a, max_jobs, (hipStream_t)stream))
                             : q8 ? bd::launch_linear_decode_tiled_q8(a, max_jobs, (hipStream_t)stream)
                                  : bd::launch_linear_decode_tiled(a, max_jobs, (hipStream_t)stream);
        if (e != hipSuccess) return BD_ERR_DEVICE;
    }
    return BD_OK;
}

}  // namespace

// ---- 8-bit round-to-nearest base ----

size_t bd_tiled_base_q8_bytes(int64_t out, int64_t in) {
    if (!tiled_shape_ok(out, in)) return 0;
    const size_t RB = (size_t)bd::tiled_row_blocks(out), KT = (size_t)bd::tiled_k_tiles(in);
    return RB * KT * bd::kTileBaseQ8Bytes + RB * bd::kTileRows * sizeof(float);
}

bd_status bd_quantize_base_q8(const uint16_t* w_f16, int64_t out, int64_t in, int8_t* q, float* scale, void* stream) {
    if (out < 0 || in < 0 || out > ((int64_t)1 << 31) - 1) return BD_ERR_SHAPE;
    if (out == 0) return BD_OK;
    if (!scale || (in > 0 && (!w_f16 || !q))) return BD_ERR_NULL;
    if (misaligned(w_f16, 2) || misaligned(scale, 4)) return BD_ERR_ALIGN;
    if (in > 0 && overlaps(q, (size_t)out * in, w_f16, (size_t)out * in * 2)) return BD_ERR_ALIAS;
    return bd::launch_quantize_rtn8(w_f16, out, in, q, scale, (hipStream_t)stream) == hipSuccess ? BD_OK : BD_ERR_DEVICE;
}

bd_status bd_tile_base_q8(const int8_t* q, const float* scale, int64_t out, int64_t in, void* wq_tiled, void* stream) {
    if (!tiled_shape_ok(out, in)) return BD_ERR_SHAPE;
    if (out == 0) return BD_OK;
    if (!scale || !wq_tiled || (in > 0 && !q)) return BD_ERR_NULL;
    if (misaligned(wq_tiled, 16) || misaligned(scale, 4)) return BD_ERR_ALIGN;
    const size_t bytes = bd_tiled_base_q8_bytes(out, in);
    if (overlaps(wq_tiled, bytes, q, (size_t)out * in) || overlaps(wq_tiled, bytes, scale, (size_t)out * 4)) return BD_ERR_ALIAS;
    return bd::launch_tile_base_q8(q, scale, out, in, (unsigned char*)wq_tiled, (hipStream_t)stream) == hipSuccess ? BD_OK
                                                                                                                  : BD_ERR_DEVICE;
}

bd_status bd_compress_q8(const int8_t* q, const float* scale, const uint16_t* w_ft_f16, int64_t out, int64_t in,
                         uint32_t* packed, float* alpha, void* workspace, size_t workspace_bytes, void* stream) {
    if (out < 0 || in < 0 || in % 32 != 0) return BD_ERR_SHAPE;
    if (!alpha) return BD_ERR_NULL;
    if (misaligned(alpha, 4)) return BD_ERR_ALIGN;
    if (out > 0 && in > 0) {
        if (!q || !scale || !w_ft_f16 || !packed) return BD_ERR_NULL;
        if (misaligned(q, 8) || misaligned(scale, 4) || misaligned(w_ft_f16, 16) || misaligned(packed, 16)) return BD_ERR_ALIGN;
        const size_t pbytes = (size_t)out * in / 8;
        if (overlaps(packed, pbytes, q, (size_t)out * in) || overlaps(packed, pbytes, w_ft_f16, (size_t)out * in * 2) ||
            overlaps(packed, pbytes, scale, (size_t)out * 4))
            return BD_ERR_ALIAS;
    }
    const size_t need = bd_workspace_bytes(BD_OP_COMPRESS, 0, out, in, 1);
    if (!workspace || workspace_bytes < need || misaligned(workspace, 256)) return BD_ERR_WORKSPACE;
    return bd::launch_compress_q8(q, scale, w_ft_f16, out, in, packed, alpha, (double*)workspace, (hipStream_t)stream) ==
                   hipSuccess
               ? BD_OK
               : BD_ERR_DEVICE;
}

bd_status bd_linear_multitenant_tiled_group_q8(int32_t n_mats, const uint16_t* x_f16, const void* const* wq_tiled,
                                               const uint32_t* const* tiled_by_mat_tenant,
                                               const float* const* alpha_by_mat, const int32_t* tenant_of_token,
                                               uint16_t* const* y_f16, int64_t T, const int64_t* out, int64_t in,
                                               int32_t n_tenants, void* stream) {
    return tiled_linear_impl(n_mats, x_f16, (const uint16_t* const*)wq_tiled, tiled_by_mat_tenant, alpha_by_mat, tenant_of_token,
                             y_f16, T, out, in, n_tenants, 1, stream, true, nullptr);
}

bd_status bd_linear_multitenant_tiled_q8(const uint16_t* x_f16, const void* wq_tiled, const uint32_t* const* tiled_by_tenant,
                                         const float* alpha_by_tenant, const int32_t* tenant_of_token, uint16_t* y_f16,
                                         int64_t T, int64_t out, int64_t in, int32_t n_tenants, void* stream) {
    const uint16_t* w = (const uint16_t*)wq_tiled;
    return tiled_linear_impl(1, x_f16, &w, tiled_by_tenant, &alpha_by_tenant, tenant_of_token, &y_f16, T, &out, in, n_tenants, 1,
                             stream, true, nullptr);
}

bd_status bd_linear_multitenant_tiled_group(int32_t n_mats, const uint16_t* x_f16, const uint16_t* const* w_tiled,
                                            const uint32_t* const* tiled_by_mat_tenant,
                                            const float* const* alpha_by_mat, const int32_t* tenant_of_token,
                                            uint16_t* const* y_f16, int64_t T, const int64_t* out, int64_t in,
                                            int32_t n_tenants, void* stream) {
    return tiled_linear_impl(n_mats, x_f16, w_tiled, tiled_by_mat_tenant, alpha_by_mat, tenant_of_token, y_f16, T, out, in,
                             n_tenants, 1, stream, false, nullptr);
}

bd_status bd_linear_multitenant_tiled(const uint16_t* x_f16, const uint16_t* w_tiled,
                                      const uint32_t* const* tiled_by_tenant, const float* alpha_by_tenant,
                                      const int32_t* tenant_of_token, uint16_t* y_f16, int64_t T, int64_t out, int64_t in,
                                      int32_t n_tenants, void* stream) {
    return tiled_linear_impl(1, x_f16, &w_tiled, tiled_by_tenant, &alpha_by_tenant, tenant_of_token, &y_f16, T, &out, in,
                             n_tenants, 1, stream, false, nullptr);
}

bd_status bd_linear_multitenant_tiled_variant(const uint16_t* x_f16, const uint16_t* w_tiled,
                                              const uint32_t* const* tiled_by_tenant, const float* alpha_by_tenant,
                                              const int32_t* tenant_of_token, uint16_t* y_f16, int64_t T, int64_t out, int64_t in,
                                              int32_t n_tenants, void* stream, int32_t variant) {
    if (variant != 0 && variant != kVariantRowMajorMfma && wide_split_of_variant(variant, in, false) < 0) return BD_ERR_UNSUPPORTED;
    return tiled_linear_impl(1, x_f16, &w_tiled, tiled_by_tenant, &alpha_by_tenant, tenant_of_token, &y_f16, T, &out, in,
                             n_tenants, 1, stream, false, nullptr, nullptr, variant);
}

bd_status bd_linear_multitenant_tiled_gemm(const uint16_t* x_f16, const uint16_t* w_tiled, const uint32_t* const* tiled_by_tenant,
                                           const float* alpha_by_tenant, const int32_t* tenant_of_token, uint16_t* y_f16,
                                           int64_t T, int64_t out, int64_t in, int32_t n_tenants, int32_t one_product,
                                           void* workspace, size_t workspace_bytes, void* stream) {
    if (T < 0 || n_tenants < 0 || T > 65535 || !tiled_shape_ok(out, in)) return BD_ERR_SHAPE;
    if ((uint64_t)T * (uint64_t)in * 2 >= ((uint64_t)1 << 32)) return BD_ERR_SHAPE;   // 32-bit byte offsets into x
    if (T == 0 || out == 0) return BD_OK;
    if (!x_f16 || !w_tiled || !tiled_by_tenant || !alpha_by_tenant || !tenant_of_token || !y_f16) return BD_ERR_NULL;
    if (misaligned(x_f16, 16) || misaligned(w_tiled, 16) || misaligned(y_f16, 2) || misaligned(alpha_by_tenant, 4)) return BD_ERR_ALIGN;
    for (int64_t t = 0; t < T; ++t) {
        const int32_t e = tenant_of_token[t];
        if (e < 0 || e >= n_tenants) return BD_ERR_TENANT;
        if (!tiled_by_tenant[e]) return BD_ERR_NULL;          // a tenant with a token needs its delta
        if (misaligned(tiled_by_tenant[e], 16)) return BD_ERR_ALIGN;
    }
    const size_t ybytes = (size_t)T * (size_t)out * 2;
    if (overlaps(y_f16, ybytes, x_f16, (size_t)T * (size_t)in * 2) || overlaps(y_f16, ybytes, w_tiled, bd_tiled_base_bytes(out, in)))
        return BD_ERR_ALIAS;
    if (in == 0 || !bd::prefill_big_fits(T, out, in)) return BD_ERR_UNSUPPORTED;   // whole k steps of 64
    const size_t need = tiled_gemm_workspace_bytes(T, n_tenants);
    if (!workspace || workspace_bytes < need || misaligned(workspace, 256)) return BD_ERR_WORKSPACE;
    return run_prefill(x_f16, w_tiled, nullptr, alpha_by_tenant, tenant_of_token, order_by_tenant(tenant_of_token, T, n_tenants), y_f16, T, out, in, workspace, (hipStream_t)stream, 4,
                       true, 0, nullptr, one_product != 0, tiled_by_tenant, n_tenants) == hipSuccess
               ? BD_OK
               : BD_ERR_DEVICE;
}

bd_status bd_linear_multitenant_tiled_group_kbit(int32_t n_mats, const uint16_t* x_f16, const uint16_t* const* w_tiled,
                                                 const uint32_t* const* planes_by_mat_tenant,
                                                 const float* const* alpha_by_mat, const int32_t* tenant_of_token,
                                                 uint16_t* const* y_f16, int64_t T, const int64_t* out, int64_t in,
                                                 int32_t n_tenants, int32_t k, void* stream) {
    return tiled_linear_impl(n_mats, x_f16, w_tiled, planes_by_mat_tenant, alpha_by_mat, tenant_of_token, y_f16, T, out, in,
                             n_tenants, k, stream, false, nullptr);
}

bd_status bd_linear_multitenant_kbit(const uint16_t* x_f16, const uint16_t* w_base_f16, const uint32_t* const* planes_by_tenant,
                                     const float* alpha_by_tenant, const int32_t* tenant_of_token, uint16_t* y_f16, int64_t T,
                                     int64_t out, int64_t in, int32_t n_tenants, int32_t k, void* stream) {
    if (k < 1 || k > bd::kTiledMaxPlanes) return BD_ERR_SHAPE;
    const bd_status st = check_linear_args(x_f16, w_base_f16, planes_by_tenant, alpha_by_tenant, tenant_of_token, y_f16, T, out, in,
                                           n_tenants);
    if (st != BD_OK) return st;
    if (T == 0 || out == 0) return BD_OK;
    // the matrix-core kernel on the row-major tensors: whole groups of four sign words, 32-bit byte offsets
    if (in % 128 != 0 || in == 0 || (uint64_t)out * (uint64_t)in * 2 >= ((uint64_t)1 << 32)) return BD_ERR_UNSUPPORTED;
    return tiled_linear_impl(1, x_f16, &w_base_f16, nullptr, &alpha_by_tenant, tenant_of_token, &y_f16, T, &out, in, n_tenants, k,
                             stream, false, planes_by_tenant);
}

// The GEMM form for any T >= 1 with k planes per tenant (128 x 128 tiles) or the 8-bit base (128 x 256 where the shape allows).
static bd_status gemm_entry(const uint16_t* x_f16, const void* w, size_t w_bytes_per_el, const uint32_t* const* packed_by_tenant,
                            const float* alpha_by_tenant, const float* wscale, const int32_t* tenant_of_token, uint16_t* y_f16,
                            int64_t T, int64_t out, int64_t in, int32_t n_tenants, int k_planes, void* workspace,
                            size_t workspace_bytes, void* stream, int32_t variant = 0) {
    const bd_status st = check_linear_args(x_f16, w, packed_by_tenant, alpha_by_tenant, tenant_of_token, y_f16, T, out, in,
                                           n_tenants, w_bytes_per_el);
    if (st != BD_OK) return st;
    const int planes = std::max(k_planes, 1);
    const int panel_split = panel_split_of_variant(variant, planes);
    if (variant != 0 && variant != kVariantPrefillSmall && variant != kVariantPrefillBig && panel_split < 0) return BD_ERR_UNSUPPORTED;
    if (T == 0 || out == 0) return BD_OK;
    if (in == 0) return BD_ERR_UNSUPPORTED;   // the empty reduction (y = 0) is bd_linear_multitenant's
    const size_t need = prefill_table_bytes(T, n_tenants);
    if (!workspace || workspace_bytes < need || misaligned(workspace, 256)) return BD_ERR_WORKSPACE;
    // The 8-bit base: 128 x 256 tiles where whole 64-wide steps and a full tile's width of output rows are there, as for fp16.
    // (k planes stay on the 128 x 128 tiles: their sums are formed in fp16 in LDS, which the large tile has no room for.)
    const bool big = wscale && k_planes == 0 && out >= 256 && bd::prefill_big_fits(T, out, in) && variant != kVariantPrefillSmall;
    if (variant == kVariantPrefillBig && !big) return BD_ERR_UNSUPPORTED;
    const bool panels = panel_fits(T, out, in, planes, wscale != nullptr);
    if (panel_split >= 0 && !panels) return BD_ERR_UNSUPPORTED;
    const std::vector<int32_t> order = order_by_tenant(tenant_of_token, T, n_tenants);
    // Few tokens per tenant, few rows: the GEMM's tiles are mostly padding and too few to fill the chip, each a serial chain of `in` / 64 steps.  The
    // panel kernel splits `in` between its wavefronts and pads to 16 tokens (us, GEMM / panels; two planes: 29 tokens of 11 tenants on 724 x 2880
    // 95 / 18, 731 of 4 on 2846 x 8960 290 / 175, 1588 of 14 on 5149 x 8960 678 / 663, 1270 of 5 on 5318 x 704 45 / 86; 8-bit base: 46 of 6 on 2884 x 7424
    // 84 / 31, 648 of 14 on 1875 x 3456 59 / 45, 717 of 5 on 4705 x 4608 106 / 117).  It is taken where its estimate is clearly the lower one.
    if (panels && (variant == 0 || panel_split >= 0)) {
        const BatchShape shape = batch_shape(tenant_of_token, order);
        const int cus = cus_or_256();
        // 0.87: the two estimates miss by about a tenth each way; at 0.9 two of 150 prompts took panels 5 and 15 % above the GEMM, at 0.87 none of 250
        if (panel_split >= 0 ||
            panel_us(shape.tiles16, out, in, cus, planes, wscale != nullptr) < 0.87 * gemm_extended_us(shape, out, in, big, planes, wscale != nullptr, cus))
            return run_wide(wide_tiles(tenant_of_token, order), x_f16, (const uint16_t*)w, packed_by_tenant, nullptr, alpha_by_tenant, y_f16, out, in,
                            (hipStream_t)stream, std::max(panel_split, 0), planes, wscale) == hipSuccess
                       ? BD_OK
                       : BD_ERR_DEVICE;
    }
    return run_prefill(x_f16, w, packed_by_tenant, alpha_by_tenant, tenant_of_token, order, y_f16, T, out, in, workspace,
                       (hipStream_t)stream, big ? 4 : 0, big, k_planes, wscale) == hipSuccess
               ? BD_OK
               : BD_ERR_DEVICE;
}

bd_status bd_linear_multitenant_gemm_kbit_variant(const uint16_t* x_f16, const uint16_t* w_base_f16,
                                                  const uint32_t* const* planes_by_tenant, const float* alpha_by_tenant,
                                                  const int32_t* tenant_of_token, uint16_t* y_f16, int64_t T, int64_t out, int64_t in,
                                                  int32_t n_tenants, int32_t k, void* workspace, size_t workspace_bytes, void* stream,
                                                  int32_t variant) {
    if (k < 1 || k > bd::kTiledMaxPlanes) return BD_ERR_SHAPE;
    return gemm_entry(x_f16, w_base_f16, 2, planes_by_tenant, alpha_by_tenant, nullptr, tenant_of_token, y_f16, T, out, in,
                      n_tenants, k, workspace, workspace_bytes, stream, variant);
}

bd_status bd_linear_multitenant_gemm_kbit(const uint16_t* x_f16, const uint16_t* w_base_f16,
                                          const uint32_t* const* planes_by_tenant, const float* alpha_by_tenant,
                                          const int32_t* tenant_of_token, uint16_t* y_f16, int64_t T, int64_t out, int64_t in,
                                          int32_t n_tenants, int32_t k, void* workspace, size_t workspace_bytes, void* stream) {
    return bd_linear_multitenant_gemm_kbit_variant(x_f16, w_base_f16, planes_by_tenant, alpha_by_tenant, tenant_of_token, y_f16, T, out,
                                                   in, n_tenants, k, workspace, workspace_bytes, stream, 0);
}

bd_status bd_linear_multitenant_gemm_q8_variant(const uint16_t* x_f16, const int8_t* q, const float* wscale,
                                                const uint32_t* const* packed_by_tenant, const float* alpha_by_tenant,
                                                const int32_t* tenant_of_token, uint16_t* y_f16, int64_t T, int64_t out, int64_t in,
                                                int32_t n_tenants, void* workspace, size_t workspace_bytes, void* stream,
                                                int32_t variant) {
    if (T > 0 && out > 0 && !wscale) return BD_ERR_NULL;
    if (misaligned(wscale, 4)) return BD_ERR_ALIGN;
    return gemm_entry(x_f16, q, 1, packed_by_tenant, alpha_by_tenant, wscale, tenant_of_token, y_f16, T, out, in, n_tenants, 0,
                      workspace, workspace_bytes, stream, variant);
}

bd_status bd_linear_multitenant_gemm_q8(const uint16_t* x_f16, const int8_t* q, const float* wscale,
                                        const uint32_t* const* packed_by_tenant, const float* alpha_by_tenant,
                                        const int32_t* tenant_of_token, uint16_t* y_f16, int64_t T, int64_t out, int64_t in,
                                        int32_t n_tenants, void* workspace, size_t workspace_bytes, void* stream) {
    return bd_linear_multitenant_gemm_q8_variant(x_f16, q, wscale, packed_by_tenant, alpha_by_tenant, tenant_of_token, y_f16, T, out, in,
                                                 n_tenants, workspace, workspace_bytes, stream, 0);
}

bd_status bd_linear_multitenant_q8(const uint16_t* x_f16, const int8_t* q, const float* wscale,
                                   const uint32_t* const* packed_by_tenant, const float* alpha_by_tenant,
                                   const int32_t* tenant_of_token, uint16_t* y_f16, int64_t T, int64_t out, int64_t in,
                                   int32_t n_tenants, void* stream) {
    const bd_status st = check_linear_args(x_f16, q, packed_by_tenant, alpha_by_tenant, tenant_of_token, y_f16, T, out, in,
                                           n_tenants, 1);
    if (st != BD_OK) return st;
    if (T == 0 || out == 0) return BD_OK;
    if (!wscale) return BD_ERR_NULL;
    if (misaligned(wscale, 4)) return BD_ERR_ALIGN;
    // the matrix-core kernel on the row-major tensors: whole groups of four sign words, 32-bit byte offsets
    if (in % 128 != 0 || in == 0 || (uint64_t)out * (uint64_t)in >= ((uint64_t)1 << 32)) return BD_ERR_UNSUPPORTED;
    const uint16_t* w = (const uint16_t*)q;
    return tiled_linear_impl(1, x_f16, &w, nullptr, &alpha_by_tenant, tenant_of_token, &y_f16, T, &out, in, n_tenants, 1, stream,
                             true, packed_by_tenant, wscale);
}

bd_status bd_linear_multitenant_tiled_kbit(const uint16_t* x_f16, const uint16_t* w_tiled,
                                           const uint32_t* const* planes_by_tenant, const float* alpha_by_tenant,
                                           const int32_t* tenant_of_token, uint16_t* y_f16, int64_t T, int64_t out,
                                           int64_t in, int32_t n_tenants, int32_t k, void* stream) {
    return tiled_linear_impl(1, x_f16, &w_tiled, planes_by_tenant, &alpha_by_tenant, tenant_of_token, &y_f16, T, &out, in,
                             n_tenants, k, stream, false, nullptr);
}

bd_status bd_group_tokens(const int32_t* tenant_of_token, int32_t T, int32_t* token_of_col, int32_t* job_tenant,
                          int32_t* job_tile, int32_t* job_col_begin, int32_t* job_col_end, int32_t* n_jobs) {
    if (T < 1 || T > kMaxDecodeTokens) return BD_ERR_SHAPE;
    if (!tenant_of_token || !token_of_col || !job_tenant || !job_tile || !job_col_begin || !job_col_end || !n_jobs)
        return BD_ERR_NULL;
    DecodeMeta m;
    build_meta(tenant_of_token, 0, T, &m);
    for (int i = 0; i < T; ++i) token_of_col[i] = m.token_of_col[i];
    for (int j = 0; j < m.n_jobs; ++j) {
        job_tenant[j] = m.job_tenant[j];
        job_tile[j] = m.job_tile[j];
        job_col_begin[j] = m.job_col_begin[j];
        job_col_end[j] = m.job_col_end[j];
    }
    *n_jobs = m.n_jobs;
    return BD_OK;
}

bd_status bd_materialize(const uint16_t* w_base_f16, const uint32_t* packed, const float* alpha, uint16_t* w_out_f16,
                         int64_t out, int64_t in, void* stream) {
    if (out < 0 || in < 0 || in % 32 != 0) return BD_ERR_SHAPE;
    if (out == 0 || in == 0) return BD_OK;
    if (!w_base_f16 || !packed || !alpha || !w_out_f16) return BD_ERR_NULL;
    if (misaligned(w_base_f16, 16) || misaligned(packed, 16) || misaligned(w_out_f16, 16)) return BD_ERR_ALIGN;
    return bd::launch_materialize(w_base_f16, packed, alpha, w_out_f16, out, in, (hipStream_t)stream) == hipSuccess
               ? BD_OK
               : BD_ERR_DEVICE;
}

bd_status bd_linear_naive(const uint16_t* x_f16, const uint16_t* const* w_by_tenant, const int32_t* tenant_of_token,
                          uint16_t* y_f16, int64_t T, int64_t out, int64_t in, int32_t n_tenants, void* stream) {
    if (T < 0 || out < 0 || in < 0 || n_tenants < 0 || in % 8 != 0 || T > 65535) return BD_ERR_SHAPE;
    if (T == 0 || out == 0) return BD_OK;
    if (!x_f16 || !w_by_tenant || !tenant_of_token || !y_f16) return BD_ERR_NULL;
    if (misaligned(x_f16, 16) || misaligned(y_f16, 2)) return BD_ERR_ALIGN;
    for (int64_t t = 0; t < T; ++t)
        if (tenant_of_token[t] < 0 || tenant_of_token[t] >= n_tenants) return BD_ERR_TENANT;
    for (int64_t t0 = 0; t0 < T; t0 += kMaxDecodeTokens) {
        const int n = (int)std::min<int64_t>(kMaxDecodeTokens, T - t0);
        DecodeMeta meta;
        build_meta(tenant_of_token, t0, n, &meta);
        if (bd::launch_linear_naive(x_f16 + t0 * in, w_by_tenant, meta, y_f16 + t0 * out, out, in,
                                    (hipStream_t)stream) != hipSuccess)
            return BD_ERR_DEVICE;
    }
    return BD_OK;
}

bd_status bd_probe_read(const void* src, size_t bytes, uint32_t* sink, void* stream) {
    if (bytes % 16 != 0) return BD_ERR_SHAPE;
    if (bytes == 0) return BD_OK;
    if (!src || !sink) return BD_ERR_NULL;
    if (misaligned(src, 16) || misaligned(sink, 4)) return BD_ERR_ALIGN;
    return bd::launch_probe_read(src, bytes, sink, (hipStream_t)stream) == hipSuccess ? BD_OK : BD_ERR_DEVICE;
}

bd_status bd_probe_copy(void* dst, const void* src, size_t bytes, void* stream) {
    if (bytes % 16 != 0) return BD_ERR_SHAPE;
    if (bytes == 0) return BD_OK;
    if (!dst || !src) return BD_ERR_NULL;
    if (misaligned(src, 16) || misaligned(dst, 16)) return BD_ERR_ALIGN;
    if (overlaps(dst, bytes, src, bytes)) return BD_ERR_ALIAS;
    return bd::launch_probe_copy(dst, src, bytes, (hipStream_t)stream) == hipSuccess ? BD_OK : BD_ERR_DEVICE;
}

}  // extern "C"

// The multi-tenant linear (Eq. 6 of the paper) on the row-major tensors for batches of tens to a few hundred tokens, a few of each tenant,
// where `out` has enough rows to fill the chip (the kernel of linear_wide.hip takes the others), for batches of up to 32 tokens that a decode
// launch would mostly wait on, and its two extensions, k sign planes per
// tenant and the 8-bit base, for prompts that are too short or matrices too small for the GEMM's tiles.
//     y[t, n] = sum_k x[t,k] W_base[n,k]  +  sum_j alpha_{e,j} * sum_k x[t,k] s_{e,j}[n,k],   e = tenant(t)
//
// As there, tokens are sorted by tenant and padded to column tiles of 16 per tenant.  There every wavefront of a workgroup has its own part
// of `in` and fetches and turns its own x: 16 KiB through the LDS for 8 KiB of table look-ups, and x passes the address unit once
// for every two row blocks (64 % of its cycles busy, the LDS 54 %, the matrix pipes 23 %).  Here a workgroup takes a panel of four row
// blocks (64 output features) and up to five column tiles; four wavefronts, one per row block, share the x of a unit of 128 k through
// LDS, and the other four do the same with the second half of `in`.  What a wavefront pays per pair of MFMAs (base and +-1 product
// of 16 features x 32 k x 16 tokens) is then one look-up and one read of x: a loop of nothing else runs at 5.0 ns per
// pair and compute unit, where the MFMAs alone take 4.2.
//
// Per iteration (one unit of 128 k for either half): one barrier, behind which x of the next unit goes from registers to the other buffer and
// that of the unit after it is requested; the base, 16 rows x 256 bytes per wavefront, is turned to operand order through a 2 KiB
// room of the wavefront's own, 64 k at a time, and requested two iterations ahead; signs come for four units at a time, 64 bytes
// of a row by four lanes side by side (16 bytes a row would be an access of its own per lane), pass through the same room and are
// turned with byte and lane shuffles.  The halves' sums are added in LDS, base and +-1 apart; alpha multiplies the finished one.
//
// Measured, weights from HBM, kernel of linear_wide.hip / this one, us: 200 tokens of 16 tenants on 4096 x 4096 54 / 34 (19 column tiles: 256 workgroups of
// 5), 400 of 32 105 / 79, 100 of 12 39 / 27, 200 of 16 on 11008 x 4096 158 / 107, 500 of 32 280 / 220, 300 of 10 on 2048 x 2048 19 / 14.  120 drawn batches
// of 33 to 700 tokens through the dispatch: 1.23 x.  What bounds it: an iteration takes 0.31 us per column tile, of which LDS accesses are 0.2 (55 % of
// the launch, address unit 52 %, matrix pipes 31 %); a ring of 2, 3, 4 or 6 pairs is the same within 2 %, and without any one of look-ups,
// reads of x, fetches of x or MFMAs it would be 5 to 17 % shorter.
// k planes and the 8-bit base, GEMM tiles / panels: 31 tokens of 11 tenants on 584 x 10624 with two planes 323 / 52, 62 of 9 on 852 x 5248 with four
// 246 / 43, 69 of 14 on 1167 x 7744 over the 8-bit base 119 / 31, 46 of 6 on 2884 x 7424 over it 96 / 30; 250 drawn prompts of 24 to 4096 tokens
// through the dispatch 1.84 x, none of them slower.
#include "bd_device.h"
#include "bd_launch.h"
#include "bd_tiled.h"

namespace bd {

namespace {

constexpr int kPanelLutBytes = 256 * 16 * 16;
constexpr int kPanelRoom = 2048;                        // per wavefront
constexpr int kPanelX = kPanelLutBytes + 8 * kPanelRoom;   // x: [buffer][half of `in`][column tile][16 rows x 256 bytes]
typedef u32x4 __attribute__((address_space(3)))* panel_lds_u32x4;
typedef const u32x2 __attribute__((address_space(3)))* panel_lds_u32x2;
typedef const u32x4 __attribute__((address_space(1)))* panel_global_u32x4;
typedef const unsigned char __attribute__((address_space(1)))* panel_global_bytes;
__device__ __forceinline__ u32x4 panel_get(const uint32_t at) { return *(panel_lds_u32x4)(uintptr_t)at; }
__device__ __forceinline__ void panel_put(const uint32_t at, const u32x4 v) { *(panel_lds_u32x4)(uintptr_t)at = v; }

__device__ __forceinline__ void panel_wave_sync() {   // a wavefront's LDS accesses run in order; this keeps the compiler's order
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ void panel_barrier() {     // orders LDS only: the global loads in flight stay in flight
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <int MT> constexpr int panel_lds_bytes() { return kPanelX + 2 * 2 * MT * 4096; }

}  // namespace

// NP sign planes per tenant, each with a +-1 sum of its own.  Q8: the base is the row-major int8 q [out, in] with a scale per row; the base
// accumulators hold sum_k x q.
template <int MT, int NP, bool Q8>
__global__ __launch_bounds__(8 * kWave) void linear_panel_kernel(const WideArgs a) {
    static_assert(panel_lds_bytes<MT>() <= 160 * 1024, "LDS budget");
    static_assert(MT <= panel_max_chunk(NP), "registers");
    extern __shared__ __align__(16) unsigned char smem[];   // starts at LDS address 0 (the host checks it)
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    const int half = wave >> 2, sub = wave & 3;
    // Workgroup -> (row blocks, chunk of column tiles).  Ids go round-robin over the 8 XCDs; the chunks of the same row blocks
    // follow each other on one XCD, so that its L2 serves the base to all of them.  The tiles are dealt to the chunks evenly.
    const int n_chunks = (a.n_tiles + a.tiles_per_chunk - 1) / a.tiles_per_chunk;
    const int per_xcd = (int)blockIdx.x >> 3;
    const int rb = (per_xcd / n_chunks * 8 + ((int)blockIdx.x & 7)) * kPanelRowBlocks + sub;
    if (rb - sub >= a.row_blocks) return;             // the grid is padded to whole groups of 8
    const int chunk = per_xcd % n_chunks;
    const int tile0 = chunk * a.n_tiles / n_chunks, n_tiles = (chunk + 1) * a.n_tiles / n_chunks - tile0;   // 1 .. MT; the surplus repeats the last one, unstored
    const uint32_t row_bytes = (uint32_t)a.in * 2u, sign_bytes = (uint32_t)a.in >> 3, w_row_bytes = (uint32_t)a.in * (Q8 ? 1u : 2u);
    // in = 64 mod 128: the last unit has two slices.  No load may reach beyond a row (the last row ends the tensor): lanes whose piece lies
    // there read the valid half of the unit.
    const int short_unit = (a.in & 64) ? a.units - 1 : -1;

    // this half's units [u0, u0 + n_u); every wavefront runs n_it iterations
    const int n_it = (a.units + 1) >> 1, u0 = half * n_it, n_u = half ? a.units - n_it : n_it;
    // what would be fetched for an iteration beyond the half: one line of a tensor's start by all lanes, so that every iteration issues
    // the same loads and the compiler can count those in flight
    auto unit_at = [&](const int it) { return it < n_u ? (uint32_t)(u0 + it) : 0u; };
    auto live = [&](const int it) { return it < n_u ? ~0u : 0u; };

    // ---- what this lane fetches.  x: rows 4 sub .. + 3 of every column tile, 16 lanes side by side, chunk q of row r at place q ^ r of the row
    const unsigned char* const xg = (const unsigned char*)a.x;
    uint32_t xoff[MT], tokv[MT];                      // tokv: the token of column c
    {
        const int row = 4 * sub + g;
#pragma unroll
        for (int ct = 0; ct < MT; ++ct) {
            const int tile = tile0 + min(ct, n_tiles - 1);
            uint32_t tok = a.col_token[tile][row];
            // an empty column reads the tile's first token: valid memory, its results are never stored
            if (tok == kWideNoToken) tok = a.col_token[tile][0];
            tokv[ct] = a.col_token[tile][c];
            xoff[ct] = tok * row_bytes + ((uint32_t)(c ^ row) << 4);
        }
    }
    const uint32_t x_back = (uint32_t)((c ^ (4 * sub + g)) & 8) << 4;   // short unit: chunks 8 .. 15 do not exist
    // base: rows 8 j .. 8 j + 7 of the row block, 8 lanes side by side (128 bytes: 64 k, 8-bit base 128 k); chunk q of row r at
    // place q ^ (r / 2 % 8)
    const unsigned char* const wg = (const unsigned char*)a.w;
    uint32_t woff[2], w_back[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int r = 8 * j + (lane >> 3);
        const int q = (lane & 7) ^ ((r >> 1) & 7);
        woff[j] = (uint32_t)min(rb * kTileRows + r, a.out - 1) * w_row_bytes + ((uint32_t)q << 4);
        w_back[j] = Q8 ? (uint32_t)(q & 4) << 4 : 0u;   // short unit of the 8-bit base: chunks 4 .. 7 do not exist
    }
    float4v wscale = {1.f, 1.f, 1.f, 1.f};            // of this lane's four features
    if constexpr (Q8) {
#pragma unroll
        for (int e = 0; e < 4; ++e) wscale[e] = a.wscale[min(rb * kTileRows + 4 * g + e, a.out - 1)];
    }
    // signs: four units of row lane / 4, 16 bytes each, by four lanes side by side
    const uint32_t soff = (uint32_t)min(rb * kTileRows + (lane >> 2), a.out - 1) * sign_bytes;
    panel_global_bytes sp[MT][NP];                    // (generic pointers would make flat loads, which LDS reads wait for)
    float alpha[MT][NP];
#pragma unroll
    for (int ct = 0; ct < MT; ++ct)
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int entry = a.tenant[tile0 + min(ct, n_tiles - 1)] * NP + j;
            alpha[ct][j] = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, a.alpha_by_tenant[entry])));
            sp[ct][j] = (panel_global_bytes)a.packed_by_tenant[entry];
        }

    constexpr int kWLoads = Q8 ? 2 : 4;
    u32x4 xs[MT], wr[2][kWLoads], sraw[MT][NP];       // as fetched
    auto ld_x = [&](const int it) __attribute__((always_inline)) {
        const unsigned char* const p = xg + (uint64_t)(unit_at(it) * 256u);
        const uint32_t back = u0 + it == short_unit ? x_back : 0u;
#pragma unroll
        for (int ct = 0; ct < MT; ++ct) {
            uint32_t o = (xoff[ct] - back) & live(it);
            asm volatile("" : "+v"(o));               // "base + lane offset" stays a 32-bit offset
            xs[ct] = *(const u32x4*)(p + o);
        }
    };
    auto ld_w = [&](u32x4 (&w)[kWLoads], const int it, const int h) __attribute__((always_inline)) {
        const bool is_short = u0 + it == short_unit;
        // (fp16: the second half of a short unit is its first one again, never multiplied; offsets stay above zero, so it is the base that
        // steps back)
        const unsigned char* const p = wg + (uint64_t)(unit_at(it) * (Q8 ? 128u : 256u) + (!Q8 && h == 1 && !is_short ? 128u : 0u));
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            uint32_t o = (woff[j] - (is_short ? w_back[j] : 0u)) & live(it);   // (w_back: bits of woff)
            asm volatile("" : "+v"(o));
            w[2 * h + j] = *(const u32x4*)(p + o);
        }
    };
    auto ld_s = [&](const int it) __attribute__((always_inline)) {   // four units from iteration `it` on; a short one's words as 2 and 3
        const int unit = min(u0 + it + (lane & 3), a.units - 1);
        const uint32_t o = (soff + (uint32_t)unit * 16u - (unit == short_unit ? 8u : 0u)) & live(it);
#pragma unroll
        for (int ct = 0; ct < MT; ++ct)
#pragma unroll
            for (int j = 0; j < NP; ++j) sraw[ct][j] = *(panel_global_u32x4)(sp[ct][j] + o);
    };
    ld_x(0);
    ld_w(wr[0], 0, 0);
    if constexpr (!Q8) ld_w(wr[0], 0, 1);
    ld_s(0);
    // the table: entry b, copy cp at 256 b + 16 cp; element e = bit e of b ? +1.0 : -1.0
    for (int q = threadIdx.x; q < 256 * 16; q += 8 * kWave) {
        const uint32_t b = (uint32_t)q >> 4;
        u32x4 e;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            e[i] = 0xBC00BC00u ^ (((b >> (2 * i)) & 1u) << 15) ^ (((b >> (2 * i + 1)) & 1u) << 31);
        panel_put((uint32_t)q * 16u, e);
    }
    const uint32_t room = kPanelLutBytes + (uint32_t)wave * kPanelRoom;
    const uint32_t x_put = kPanelX + (uint32_t)half * (MT * 4096u) + (uint32_t)sub * 1024u + (uint32_t)lane * 16u;
    const uint32_t x_get = kPanelX + (uint32_t)half * (MT * 4096u) + (uint32_t)c * 256u + ((uint32_t)(c ^ g) << 4);   // chunk 4 v + g: ^ 64 v
    const uint32_t w_get = room + (uint32_t)c * 128u + ((uint32_t)(g ^ ((c >> 1) & 7)) << 4);                         // chunk 4 v + g: ^ 64 v
    const uint32_t q_get = room + (uint32_t)c * 128u + ((uint32_t)((g >> 1) ^ ((c >> 1) & 7)) << 4) + (uint32_t)(g & 1) * 8u;   // chunk 2 v + g / 2: ^ 32 v
    const uint32_t lanebits = (uint32_t)c << 4;
    auto put_x = [&](const int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int ct = 0; ct < MT; ++ct) panel_put(x_put + buf * (2 * MT * 4096) + ct * 4096, xs[ct]);
    };
    put_x(0);
    ld_x(1);
    ld_w(wr[1], 1, 0);
    if constexpr (!Q8) ld_w(wr[1], 1, 1);

    float4v acc[MT], dsum[MT][NP];                    // base product, +-1 sums
    u32x4 sg[MT][NP];                                 // signs of the column tiles: word j = this lane's bytes of unit j of the four
#pragma unroll
    for (int ct = 0; ct < MT; ++ct) {
        acc[ct] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < NP; ++j) dsum[ct][j] = float4v{0.f, 0.f, 0.f, 0.f};
    }

    auto iteration = [&](auto j_tag, const int it) __attribute__((always_inline)) {
        constexpr int J = decltype(j_tag)::value, P = J & 1;
        put_x(P ^ 1);
        ld_x(it + 2);
        if constexpr (J == 0) {
            const bool mine = min(u0 + it + (lane & 3), a.units - 1) == short_unit;   // this lane's piece is the short unit's
#pragma unroll
            for (int ct = 0; ct < MT; ++ct)
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    u32x4 w = sraw[ct][j];
                    w[0] = mine ? w[2] : w[0];
                    w[1] = mine ? w[3] : w[1];
                    panel_wave_sync();
                    panel_put(room + (uint32_t)lane * 16u, w);
                    panel_wave_sync();
                    sg[ct][j] = panel_get(room + (uint32_t)c * 64u + (uint32_t)g * 16u);
                }
#pragma unroll
            for (int ct = 0; ct < MT; ++ct)
#pragma unroll
                for (int j = 0; j < NP; ++j) sg[ct][j] = turn_sign_words(sg[ct][j]);
            ld_s(it + 4);
        }
        u32x4 wo[4];
        auto turn_w = [&](const int h) __attribute__((always_inline)) {   // 64 k; 8-bit base: h = 0 turns all 128
            if (Q8 && h == 1) return;
            panel_wave_sync();
#pragma unroll
            for (int j = 0; j < 2; ++j) panel_put(room + j * 1024u + (uint32_t)lane * 16u, wr[P][(Q8 ? 0 : 2 * h) + j]);
            panel_wave_sync();
            if constexpr (Q8) {
                // 8 bytes of slice v: chunk 2 v + g / 2, half g % 2.  u = q + 128 next to 0x64 is the fp16 number 1024 + u, minus 1152 it is q exactly
                const half2v off = half2v{(_Float16)1152.f, (_Float16)1152.f};
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const u32x2 b = *(panel_lds_u32x2)(uintptr_t)(q_get ^ (32u * v));
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const uint32_t u = b[i >> 1] ^ 0x80808080u;
                        wo[v][i] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(half2v, __builtin_amdgcn_perm(0x64646464u, u, (i & 1) ? 0x04030402u : 0x04010400u)) - off);
                    }
                }
            } else {
#pragma unroll
                for (int v = 0; v < 2; ++v) wo[2 * h + v] = panel_get(w_get ^ (64u * v));
            }
            ld_w(wr[P], it + 2, h);
        };
        turn_w(0);
        // step n of the unit: half h of its 128 k, column tile, slice
        // (three planes and three column tiles: with two ahead two registers went to scratch, and such prompts took 2 to 5 % longer:
        // 14 tokens of 3 tenants on 11533 x 1152 19.5 / 18.7 us, 90 of 7 on 10813 x 960 40.9 / 39.0)
        constexpr int kSteps = 4 * MT, kAhead = NP == 1 ? 3 : NP == 3 && MT == 3 ? 1 : 2, kRing = kAhead + 1;
        u32x4 lut[kRing][NP], xo[kRing];
        auto look_up = [&](const int n) __attribute__((always_inline)) {
            const int h = n / (2 * MT), ct = n % (2 * MT) / 2, v = 2 * h + (n & 1);
#pragma unroll
            for (int j = 0; j < NP; ++j)
                lut[n % kRing][j] = panel_get(__builtin_amdgcn_perm(sg[ct][j][J], lanebits, 0x0C0C0000u | ((4u + v) << 8)));
            xo[n % kRing] = panel_get((x_get ^ (64u * v)) + P * (2 * MT * 4096) + ct * 4096);
        };
        auto step = [&](const int n) __attribute__((always_inline)) {
            const int h = n / (2 * MT), ct = n % (2 * MT) / 2, v = 2 * h + (n & 1);
            if (n + kAhead < kSteps) look_up(n + kAhead);
            const half8 xv = __builtin_bit_cast(half8, xo[n % kRing]);
            acc[ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, wo[v]), xv, acc[ct], 0, 0, 0);
#pragma unroll
            for (int j = 0; j < NP; ++j)
                dsum[ct][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, lut[n % kRing][j]), xv, dsum[ct][j], 0, 0, 0);
            if (n == 2 * MT - 3) turn_w(1);
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int n = 0; n < kAhead; ++n) look_up(n);
#pragma unroll
        for (int n = 0; n < 2 * MT; ++n) step(n);
        if (u0 + it == short_unit) return;
#pragma unroll
        for (int n = 2 * MT; n < kSteps; ++n) step(n);
    };
    // A barrier begins an iteration: x of this unit is in its buffer, and nobody reads the other one any more.  (The second half may have a
    // unit less: its wavefronts leave at the last barrier.)
    for (int it = 0;;) {
        panel_barrier();
        if (it >= n_u) break;
        iteration(std::integral_constant<int, 0>{}, it);
        if (++it == n_it) break;
        panel_barrier();
        if (it >= n_u) break;
        iteration(std::integral_constant<int, 1>{}, it);
        if (++it == n_it) break;
        panel_barrier();
        if (it >= n_u) break;
        iteration(std::integral_constant<int, 2>{}, it);
        if (++it == n_it) break;
        panel_barrier();
        if (it >= n_u) break;
        iteration(std::integral_constant<int, 3>{}, it);
        if (++it == n_it) break;
    }

    // ---- the second half's sums to the first half's wavefronts: [sub][ct][base, +-1 of the planes][column][row]
    __syncthreads();                                  // table and x are no longer read
    constexpr uint32_t kSums = (1 + NP) * 1024;
    const uint32_t at = (uint32_t)sub * (MT * kSums) + (uint32_t)(c * 16 + 4 * g) * 4u;
    if (half) {
#pragma unroll
        for (int ct = 0; ct < MT; ++ct) {
            *(float4v*)(smem + at + ct * kSums) = acc[ct];
#pragma unroll
            for (int j = 0; j < NP; ++j) *(float4v*)(smem + at + ct * kSums + (1 + j) * 1024) = dsum[ct][j];
        }
    }
    __syncthreads();
    if (half) return;
    const bool whole = (a.out & 3) == 0 && ((uintptr_t)a.y & 7) == 0;
    const int n = rb * kTileRows + 4 * g;             // this lane: four features of the token of column c
#pragma unroll
    for (int ct = 0; ct < MT; ++ct) {
        if (ct >= n_tiles) continue;
        const uint32_t tok = tokv[ct];
        float4v sum = acc[ct] + *(const float4v*)(smem + at + ct * kSums);
        if constexpr (Q8) {
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] *= wscale[e];
        }
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const float4v d = dsum[ct][j] + *(const float4v*)(smem + at + ct * kSums + (1 + j) * 1024);
#pragma unroll
            for (int e = 0; e < 4; ++e) sum[e] += alpha[ct][j] * d[e];
        }
        if (tok == kWideNoToken || n >= a.out) continue;
        uint16_t h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) h[e] = f2h_rne(sum[e]);
        uint16_t* const y = a.y + (int64_t)tok * a.out + n;
        if (whole) {
            *(u32x2*)y = u32x2{(uint32_t)h[0] | (uint32_t)h[1] << 16, (uint32_t)h[2] | (uint32_t)h[3] << 16};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < a.out) y[e] = h[e];
        }
    }
}

template <int MT, int NP, bool Q8>
static hipError_t launch_panel_inst(const WideArgs& args, hipStream_t st) {
    auto kernel = linear_panel_kernel<MT, NP, Q8>;
    constexpr int lds = panel_lds_bytes<MT>();
    static PerDeviceOnce once;
    const hipError_t ea = once.run([&] {
        hipFuncAttributes fa;
        const hipError_t e = hipFuncGetAttributes(&fa, (const void*)kernel);
        if (e != hipSuccess) return e;
        if (fa.sharedSizeBytes != 0) return hipErrorInvalidValue;   // the table must start at LDS address 0
        return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    });
    if (ea != hipSuccess) return ea;
    const unsigned groups = (unsigned)((args.row_blocks + kPanelRowBlocks - 1) / kPanelRowBlocks);
    const unsigned chunks = (unsigned)((args.n_tiles + args.tiles_per_chunk - 1) / args.tiles_per_chunk);
    hipLaunchKernelGGL(kernel, dim3((groups + 7) / 8 * 8 * chunks), dim3(8 * kWave), lds, st, args);
    return hipGetLastError();
}

// args.n_tiles column tiles (1 .. kWideMaxTiles) in chunks of at most args.tiles_per_chunk (1 .. panel_max_chunk(planes)); planes 1 .. kPanelMaxPlanes,
// wscale with one plane only
hipError_t launch_linear_panel(const WideArgs& args, int planes, hipStream_t st) {
    const int n = args.tiles_per_chunk;
    if (planes < 1 || planes > kPanelMaxPlanes || args.n_tiles < 1 || args.n_tiles > kWideMaxTiles || n < 1 || n > panel_max_chunk(planes) || args.in < 128 ||
        args.in % 64 != 0 || args.units != (args.in + 127) / 128 || args.out < 1 || args.row_blocks != (args.out + kTileRows - 1) / kTileRows ||
        !args.packed_by_tenant || (args.wscale && planes != 1))
        return hipErrorInvalidValue;
    auto go = [&](auto np_tag, auto q8_tag) {
        constexpr int NP = decltype(np_tag)::value;
        constexpr bool Q8 = decltype(q8_tag)::value;
        if (n <= 2) return launch_panel_inst<2, NP, Q8>(args, st);
        if constexpr (panel_max_chunk(NP) >= 3) {
            if (n == 3) return launch_panel_inst<3, NP, Q8>(args, st);
        }
        if constexpr (panel_max_chunk(NP) >= 4) {
            if (n == 4) return launch_panel_inst<4, NP, Q8>(args, st);
        }
        if constexpr (panel_max_chunk(NP) >= 5) return launch_panel_inst<5, NP, Q8>(args, st);
        return hipErrorInvalidValue;
    };
    if (args.wscale) return go(std::integral_constant<int, 1>{}, std::true_type{});
    if (planes == 1) return go(std::integral_constant<int, 1>{}, std::false_type{});
    if (planes == 2) return go(std::integral_constant<int, 2>{}, std::false_type{});
    if (planes == 3) return go(std::integral_constant<int, 3>{}, std::false_type{});
    return go(std::integral_constant<int, 4>{}, std::false_type{});
}

}  // namespace bd

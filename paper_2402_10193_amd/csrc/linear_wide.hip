// The multi-tenant linear (Eq. 6 of the paper) for batches between a decode launch and a prefill GEMM: tens to a few
// hundred tokens, a few of each tenant (drafted tokens to verify, short prompts among decode tokens), and for up to 32 tokens where rows are few or
// short.  Row-major batches with rows enough for panels of 64 take the kernel of linear_panel.hip.
//     y[t, n] = sum_k x[t,k] W_base[n,k]  +  alpha_e * sum_k x[t,k] s_e[n,k],   e = tenant(t)
//
// A decode launch takes 32 tokens and streams the base once per launch; a GEMM tile of 64 or 128 rows holds one tenant's
// tokens only.  Here tokens are sorted by tenant and padded to columns of 16 per tenant (one MFMA tile), and a workgroup
// multiplies R row blocks of 16 output features with up to MT such column tiles, so the base is read once per MT tiles, a
// delta once, and a token costs at most 15 columns of padding.
//
// Decomposition.  The products are too small to fill the chip with output tiles, so the 8 wavefronts of a workgroup split
// `in` (units of 128) and their partial tiles are added in LDS in a fixed order.  Wavefronts share nothing inside the loop,
// so there is no barrier in it.  Per unit and column tile a wavefront runs 8 R MFMAs (v_mfma_f32_16x16x32_f16, A = 16
// features x 32 k, B = 32 k x 16 tokens) and fetches 4 KiB of x.  In operand order neighbouring lanes are different tokens,
// every lane an access of its own, and the address unit takes 64 cycles per KiB; so x is fetched with 16 lanes side by side
// in a row (16 cycles) and turned round through LDS rows that belong to the wavefront (16-byte chunk q of row r at place
// q ^ r: neither the writes nor the reads share a bank).  Row-major bases take the same way.  200 tokens of 16 tenants on
// 4096 x 4096, weights from HBM: 54 us on either layout; decode launches 137 (row-major) and 123 (tiled), the GEMM of 32-row
// tiles 76.  What is left: some 4 us around the loop of a workgroup, and in it the issue of two wavefronts per SIMD.
// R = 2 halves the fetches of x per product; R = 1 where two row blocks per workgroup would leave compute units idle.
//
// The sums.  Base product and +-1 sum have accumulators of their own, and a scale never multiplies an unfinished sum inside
// the loop.  (With one set of accumulators, the +-1 sum of each unit scaled and added to the base product, eight column tiles and two
// row blocks fit the registers and 400 tokens of 32 tenants took 100 us where it is 105 now; but where the +-1 sums of units
// cancel, the result then carried the rounding of alpha times the parts, and an infinite scale made an infinity of a sum of zero.)
//   Row-major: the wavefronts' sums are added, base and +-1 apart, and alpha multiplies the finished one, as in the GEMM.
//   Tiled: the arithmetic of the decode kernel, addition for addition (its k tiles per wavefront, the +-1 sum of a k tile from
//   zero and then added to those before it, the wavefronts' scaled parts in order), so that a token's result does not depend on
//   which of the two the batch was given to.  Fewer k tiles than wavefronts: the workgroup takes 2, 4 or 8 times the row blocks
//   (237 tokens of 13 tenants on 1676 x 768, where the decode kernel deals three k tiles to two wavefronts: 11 us, 21 with six idle).
// Registers (two wavefronts per SIMD, 256 each): accumulators 8 R MT, tiled 12 R MT where wavefronts have several k tiles; the base
// of two units 32 R, x 32, two table operands 8, the signs of a unit R MT.  That sets the most column tiles (wide_max_chunk).
// Signs become operands through the byte table of the decode kernel (256 entries x 16 copies x 16 B in LDS, one
// v_perm_b32 and one ds_read_b128 per 8 signs and lane).
#include "bd_device.h"
#include "bd_launch.h"
#include "bd_tiled.h"

namespace bd {

namespace {

constexpr int kWideUnit = 128;                        // reduction elements per unit: 4 MFMA slices
constexpr int kWideLutBytes = 256 * 16 * 16;
typedef const u32x4 __attribute__((address_space(3)))* wide_lds_u32x4;
typedef const u32x4 __attribute__((address_space(1)))* wide_global_u32x4;

__device__ __forceinline__ void wide_wave_sync() {   // a wavefront's LDS accesses run in order; this keeps the compiler's order
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// LDS: the table, two 4 KiB rooms per wavefront in which 16 rows x 128 k change their order; the partial tiles of eight
// wavefronts and one more set overlay both after the loop.  Behind them what is looked up per column tile.
template <int R, int MT>
struct WideLds {
    static constexpr int kRooms = kWideLutBytes;
    static constexpr int kRed = 9 * R * MT * 1024;
    static constexpr int kOff = kWideLutBytes + kWideWaves * 8192;   // [ct][lane group][i]: byte offset of x row 4 i + group
    static constexpr int kTok = kOff + MT * 64;                      // [ct][column]: token or -1
    static constexpr int kGroups = (R * MT + 3) / 4;                 // row-major signs are fetched four (ct, row block) at a time
    static constexpr int kSp = kTok + MT * 64;                       // [group][lane]: address of the lane's row of signs
    static constexpr int kAlpha = kSp + kGroups * 512;               // [ct]: the scale
    static constexpr int kTotal = kAlpha + MT * 4;
    static_assert(kRed <= kOff, "the partial tiles overlay the table and the rooms only");
};

}  // namespace

// TILE_SUMS: the +-1 sum of every pair of units (a k tile) apart
template <int R, int MT, bool RM, bool TILE_SUMS>
__global__ __launch_bounds__(kWideWaves * kWave) void linear_wide_kernel(const WideArgs a) {
    using Lds = WideLds<R, MT>;
    constexpr int kGroups = Lds::kGroups;
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int c = lane & 15, g = lane >> 4;
    // Workgroup -> (row blocks, chunk of column tiles).  Ids go round-robin over the 8 XCDs; the chunks of the same row blocks
    // follow each other on one XCD, so that its L2 serves the base to all of them.
    const int n_chunks = (a.n_tiles + a.tiles_per_chunk - 1) / a.tiles_per_chunk;
    const int per_xcd = (int)blockIdx.x >> 3;
    // Tiled: the k tiles are dealt to nw wavefronts (wide_k_waves); where that is fewer than eight, the workgroup takes `subs` times as
    // many row blocks and the wavefronts of a SIMD are on different parts of `in`.
    const int nw = RM ? kWideWaves : wide_k_waves(a.KT), subs = RM ? 1 : kWideWaves / nw;
    const int k_part = wave / subs, sub = wave % subs;
    const int rb_first = ((per_xcd / n_chunks) * 8 + ((int)blockIdx.x & 7)) * (R * subs);
    const int rb0 = rb_first + sub * R;
    const int tile0 = (per_xcd % n_chunks) * a.tiles_per_chunk;
    if (rb_first >= a.row_blocks) return;             // the grid is padded to whole groups of 8
    const int n_tiles = min(a.tiles_per_chunk, a.n_tiles - tile0);   // 1 .. MT; the surplus repeats the last one, unstored
    const uint32_t row_bytes = (uint32_t)a.in * 2u;

    // ---- per column tile: tokens, offsets of their rows, (row-major) addresses of the signs
    if (threadIdx.x < MT * 16) {
        const int ct = threadIdx.x >> 4, tile = tile0 + min(ct, n_tiles - 1);
        const uint32_t tok = a.col_token[tile][c];
        *(int*)(smem + Lds::kTok + threadIdx.x * 4) = (ct < n_tiles && tok != kWideNoToken) ? (int)tok : -1;
        // an empty column reads the tile's first token: valid memory, its results are never stored
        const uint32_t off = (tok != kWideNoToken ? tok : (uint32_t)a.col_token[tile][0]) * row_bytes;
        *(uint32_t*)(smem + Lds::kOff + ct * 64 + (c & 3) * 16 + (c >> 2) * 4) = off;
    }
    if constexpr (RM) {
        for (int q = threadIdx.x; q < kGroups * 64; q += kWideWaves * kWave) {   // lane (c, j) of group p: row c of pair f = 4 p + j
            const int f = min(4 * (q >> 6) + ((q >> 4) & 3), R * MT - 1);
            const int row = min((rb0 + f % R) * kTileRows + (q & 15), a.out - 1);   // rows beyond `out` read the last one; never stored
            const unsigned char* p = (const unsigned char*)a.packed_by_tenant[a.tenant[tile0 + min(f / R, n_tiles - 1)]];
            *(uint64_t*)(smem + Lds::kSp + q * 8) = (uint64_t)(p + (int64_t)row * (a.in >> 3));
        }
    }
    const unsigned char* sp[MT];
#pragma unroll
    for (int ct = 0; ct < MT; ++ct) {
        const int tile = tile0 + min(ct, n_tiles - 1);
        const float al = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, a.alpha_by_tenant[a.tenant[tile]])));
        if (threadIdx.x == 0) *(float*)(smem + Lds::kAlpha + ct * 4) = al;
        sp[ct] = RM ? nullptr : (const unsigned char*)a.signs[tile];
    }
    const unsigned char* const xg = (const unsigned char*)a.x;
    const unsigned char* const wg = (const unsigned char*)a.w;
    // This wavefront's units.  Row-major: every 8th, so that the 16-byte pieces of a 128-byte line of signs are asked for by
    // the 8 wavefronts at about the same time.  Tiled: those of a contiguous range of k tiles (256 elements), the range that the decode
    // kernel deals to a wavefront.
    int u_begin = wave, u_half = kWideWaves, u_step = 2 * kWideWaves, u_count = (a.units - wave + kWideWaves - 1) / kWideWaves;
    if constexpr (!RM) {
        u_begin = 2 * (k_part * a.KT / nw);
        u_half = 1;
        u_step = 2;
        u_count = min(2 * ((k_part + 1) * a.KT / nw), a.units) - u_begin;
    }

    // the table: entry b, copy cp at 256 b + 16 cp; element e = bit e of b ? +1.0 : -1.0
    for (int q = threadIdx.x; q < 256 * 16; q += kWideWaves * kWave) {
        const uint32_t b = (uint32_t)q >> 4;
        u32x4 e;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            e[i] = 0xBC00BC00u ^ (((b >> (2 * i)) & 1u) << 15) ^ (((b >> (2 * i + 1)) & 1u) << 31);
        *(u32x4*)(smem + q * 16) = e;
    }
    __syncthreads();
    const uint32_t lanebits = (uint32_t)c << 4;

    // A room: 16 rows of 256 bytes, chunk q of row r at place q ^ r.  Fetch i of a block covers rows 4 i .. 4 i + 3, 16 lanes a
    // row; the operand of slice v is chunk 4 v + g of row c.
    unsigned char* const room = smem + Lds::kRooms + wave * 8192;
    const uint32_t cg16 = (uint32_t)(c ^ g) << 4;     // (c ^ (4 i + g)) * 16 = cg16 ^ 64 i
    auto room_get = [&](const int v) __attribute__((always_inline)) {
        uint32_t l = (uint32_t)c * 256u + cg16;
        asm volatile("" : "+v"(l));                   // one register, an xor per use: four of them do not fit
        return l ^ (64u * v);
    };
    auto chunk16 = [&](const int i) __attribute__((always_inline)) {
        uint32_t l = cg16;
        asm volatile("" : "+v"(l));
        return l ^ (64u * i);
    };
    // the offsets of a tile's rows are read a tile ahead: waiting for them would drain the table look-ups in flight
    auto ld_off = [&](const int ct) __attribute__((always_inline)) { return *(const u32x4*)(smem + Lds::kOff + ct * 64 + g * 16); };
    auto ld_x = [&](u32x4 (&st)[4], const int u, const u32x4 off) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) st[i] = *(const u32x4*)(xg + (uint64_t)((uint32_t)u * 256u) + (off[i] + chunk16(i)));
    };
    // the base of one row block and unit: row-major as 16 rows x 256 bytes, tiled in operand order
    auto ld_w = [&](const int u, const int r, const int i) __attribute__((always_inline)) {
        if constexpr (RM) {
            uint32_t row = (uint32_t)min((rb0 + r) * kTileRows + 4 * i + g, a.out - 1);
            asm volatile("" : "+v"(row));             // not hoisted: eight offsets would live in registers
            return *(const u32x4*)(wg + (uint64_t)((uint32_t)u * 256u) + (row * row_bytes + chunk16(i)));
        } else {
            const uint32_t rb = (uint32_t)min(rb0 + r, a.row_blocks - 1);
            uint32_t l = (uint32_t)lane * 16u;
            asm volatile("" : "+v"(l));
            return *(const u32x4*)(wg + (uint64_t)(rb * (uint32_t)a.KT * (uint32_t)kTileBaseBytes + (uint32_t)u * 4096u + i * 1024u) + l);
        }
    };
    auto turn = [&](u32x4 (&st)[4], unsigned char* to) __attribute__((always_inline)) {   // fetched rows -> operands, in place
        wide_wave_sync();
#pragma unroll
        for (int i = 0; i < 4; ++i) *(u32x4*)(to + lane * 16 + 1024 * i) = st[i];
        wide_wave_sync();
#pragma unroll
        for (int v = 0; v < 4; ++v) st[v] = *(const u32x4*)(to + room_get(v));
    };
    // tiled: 4 sign bytes of (row block, unit) and lane
    auto ld_s = [&](const int u, const int r, const int ct) __attribute__((always_inline)) {
        const uint32_t rb = (uint32_t)min(rb0 + r, a.row_blocks - 1);
        uint32_t l = (uint32_t)lane * 8u;
        asm volatile("" : "+v"(l));
        return *(const uint32_t*)(sp[ct] + (uint64_t)(rb * (uint32_t)a.KT * (uint32_t)kTileSignBytes + (uint32_t)(u >> 1) * 512u + (uint32_t)(u & 1) * 4u) + l);
    };
    // row-major: lane (c, j) of group p fetches the 16 bytes that row c of pair f = 4 p + j has for the unit
    auto ld_s4 = [&](const int u, const int p) __attribute__((always_inline)) {
        const uint64_t ptr = *(const uint64_t*)(smem + Lds::kSp + p * 512 + lane * 8);
        return *(const wide_global_u32x4)(ptr + (uint32_t)u * 16u);   // (a generic pointer would make it a flat load, which LDS reads wait for)
    };
    float4v acc[R][MT], dsum[R][MT];                   // base product, +-1 sum
    float4v dtile[TILE_SUMS ? R : 1][TILE_SUMS ? MT : 1];   // +-1 sum of the k tile that is being multiplied
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int ct = 0; ct < MT; ++ct) acc[r][ct] = dsum[r][ct] = float4v{0.f, 0.f, 0.f, 0.f};

    u32x4 wr[2][R][4];                                 // the base of this unit and of the next one
    u32x4 xs[4], xo[4];                                // x of the next column tile as fetched; this one's operands
    u32x4 sg[kGroups];                                 // signs of pair f = ct R + r: sg[f / 4][f % 4]
    if (u_count > 0) {
        u32x4 x0[4];
        ld_x(x0, u_begin, ld_off(0));
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int i = 0; i < 4; ++i) wr[0][r][i] = ld_w(u_begin, r, i);
        if constexpr (RM) {
#pragma unroll
            for (int p = 0; p < kGroups; ++p) sg[p] = ld_s4(u_begin, p);
        } else {
#pragma unroll
            for (int f = 0; f < R * MT; ++f) sg[f / 4][f % 4] = ld_s(u_begin, f % R, f / R);
        }
        ld_x(xs, u_begin, ld_off(1));
        turn(x0, room);
#pragma unroll
        for (int v = 0; v < 4; ++v) xo[v] = x0[v];
        if constexpr (RM) {
#pragma unroll
            for (int r = 0; r < R; ++r) turn(wr[0][r], room);
        }
    }
    u32x4 off_next = ld_off(2 % MT);                   // rows of the tile that is requested next
    constexpr int kPer = 4 * R;                        // (slice, row block) pairs of a column tile
    constexpr int kAhead = 2;                          // table operands in flight (3, 4, 6 and 8 are not faster)
    static_assert(kAhead <= MT * kPer, "the first operands belong to one unit");
    u32x4 ring[kAhead];
    auto look_up = [&](const uint32_t s, const int v) __attribute__((always_inline)) {
        const uint32_t addr = __builtin_amdgcn_perm(s, lanebits, 0x0C0C0000u | ((4u + v) << 8));
        return *(wide_lds_u32x4)(uintptr_t)addr;
    };

    // table operand of pair n (= 4 R ct + R v + r) of the unit
    auto look_up_pair = [&](const int n, const int u_next) __attribute__((always_inline)) {
        const int ct = n / kPer, v = n % kPer / R, r = n % R, f = ct * R + r;
        if (RM && f % 4 == 0 && v == 0) sg[f / 4] = turn_sign_words(sg[f / 4]);
        ring[n % kAhead] = look_up(sg[f / 4][f % 4], v);
        if (v == 3) {                                  // its last look-up has been issued: the next unit's
            if constexpr (RM) {
                if (f % 4 == 3 || f == R * MT - 1) sg[f / 4] = ld_s4(u_next, f / 4);
            } else {
                sg[f / 4][f % 4] = ld_s(u_next, r, ct);
            }
        }
    };
    // One unit: all column tiles against this unit's R x 4 slices of the base (register set B).  u_next: the unit whose
    // operands are requested as registers fall free (the last unit requests itself again).
    auto unit = [&](auto b_tag, const int u, const int u_next) __attribute__((always_inline)) {
        constexpr int B = decltype(b_tag)::value;
#pragma unroll
        for (int n = 0; n < kAhead; ++n) look_up_pair(n, u_next);
#pragma unroll
        for (int ct = 0; ct < MT; ++ct) {
            // the next tile's x into the other room, and the one after it requested
            unsigned char* const to = room + ((B * MT + ct + 1) & 1) * 4096;
            wide_wave_sync();
#pragma unroll
            for (int i = 0; i < 4; ++i) *(u32x4*)(to + lane * 16 + 1024 * i) = xs[i];
            wide_wave_sync();
            ld_x(xs, ct + 2 < MT ? u : u_next, off_next);
            off_next = ld_off((ct + 3) % MT);
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int v = i / R, r = i % R;
                const half8 xv = __builtin_bit_cast(half8, xo[v]);
                acc[r][ct] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, wr[B][r][v]), xv, acc[r][ct], 0, 0, 0);
                const float4v zero = {0.f, 0.f, 0.f, 0.f};
                float4v& d = TILE_SUMS ? dtile[TILE_SUMS ? r : 0][TILE_SUMS ? ct : 0] : dsum[r][ct];
                d = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, ring[(ct * kPer + i) % kAhead]), xv,
                                                           TILE_SUMS && B == 0 && v == 0 ? zero : d, 0, 0, 0);
                if (ct * kPer + i + kAhead < MT * kPer) look_up_pair(ct * kPer + i + kAhead, u_next);
                if (r == R - 1) xo[v] = *(const u32x4*)(to + room_get(v));   // slice v has met its last row block
                // the next unit's base, dealt over this unit's pairs
                {
                    constexpr int kAll = 4 * R, kSlots = MT * kPer;
                    const int slot = ct * kPer + i;
#pragma unroll
                    for (int q = (slot * kAll + kSlots - 1) / kSlots; q < ((slot + 1) * kAll + kSlots - 1) / kSlots; ++q)
                        wr[B ^ 1][q % R][q / R] = ld_w(u_next, q % R, q / R);
                }
                // the previous tile's +-1 sums have left the matrix cores: add them up
                if constexpr (TILE_SUMS) {
                    if (B == 1 && ct > 0 && i >= kPer - R) dsum[r][ct - 1] += dtile[r][ct - 1];
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if constexpr (TILE_SUMS && B == 1) {
#pragma unroll
            for (int r = 0; r < R; ++r) dsum[r][MT - 1] += dtile[r][MT - 1];
        }
        // a row-major base: fetched rows -> operands, through the room that the next tile is not in
        if constexpr (RM) {
            unsigned char* const to = room + ((B * MT + MT + 1) & 1) * 4096;
#pragma unroll
            for (int r = 0; r < R; ++r) turn(wr[B ^ 1][r], to);
        }
    };
    {
        int k = 0, u = u_begin;
        for (; k + 1 < u_count; k += 2, u += u_step) {
            unit(std::integral_constant<int, 0>{}, u, u + u_half);
            unit(std::integral_constant<int, 1>{}, u + u_half, k + 2 < u_count ? u + u_step : u + u_half);
        }
        if (k < u_count) {                             // the half k tile that ends a row
            unit(std::integral_constant<int, 0>{}, u, u);
            if constexpr (TILE_SUMS) {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int ct = 0; ct < MT; ++ct) dsum[r][ct] += dtile[r][ct];
            }
        }
    }

    // ---- the wavefronts' partial tiles are added and written: [r][ct][column][row], a set of them is kSet bytes
    constexpr int kSet = R * MT * 1024;
    const int lane_at = (c * 16 + 4 * g) * 4;
    auto put = [&](const int at, auto value) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int ct = 0; ct < MT; ++ct) *(float4v*)(smem + at + lane_at + (r * MT + ct) * 1024) = value(r, ct);
    };
    auto scale_of = [&](const int ct) { return *(const float*)(smem + Lds::kAlpha + ct * 4); };
    // y of the row blocks of subs [s0, s0 + n_s), whose parts are in LDS; finished: infinite scales multiply the sum at 8 kSet
    const bool whole = (a.out & 3) == 0 && ((uintptr_t)a.y & 7) == 0;
    auto write_y = [&](const int s0, const int n_s, const bool finished) __attribute__((always_inline)) {
        const int per = n_tiles * 16 * (R * 4);
        for (int idx = threadIdx.x; idx < n_s * per; idx += kWideWaves * kWave) {   // four features of a token each
            const int s = RM ? 0 : s0 + idx / per, i = RM ? idx : idx % per;
            const int row = i % (R * 4) * 4, col = i / (R * 4);   // consecutive threads: consecutive features
            const int tok = *(const int*)(smem + Lds::kTok + col * 4);
            const int n = (rb_first + s * R) * kTileRows + row;
            if (tok < 0 || n >= a.out) continue;
            const unsigned char* const p = smem + ((row >> 4) * MT + (col >> 4)) * 1024 + ((col & 15) * 16 + (row & 15)) * 4;
            const float al = scale_of(col >> 4);
            float4v sum = {0.f, 0.f, 0.f, 0.f}, t = {0.f, 0.f, 0.f, 0.f};
            if constexpr (RM) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    sum += *(const float4v*)(p + 2 * w * kSet);
                    t += *(const float4v*)(p + (2 * w + 1) * kSet);
                }
            } else {
                for (int w = 0; w < nw; ++w) sum += *(const float4v*)(p + (w * subs + s) * kSet);
                if (finished) t = *(const float4v*)(p + 8 * kSet);
            }
            uint16_t h[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = f2h_rne(RM || (finished && __builtin_isinf(al)) ? sum[e] + al * t[e] : sum[e]);
            uint16_t* const y = a.y + (int64_t)tok * a.out + n;
            if (whole) {
                *(u32x2*)y = u32x2{(uint32_t)h[0] | (uint32_t)h[1] << 16, (uint32_t)h[2] | (uint32_t)h[3] << 16};
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (n + e < a.out) y[e] = h[e];
            }
        }
    };
    __syncthreads();                                   // the table is no longer read
    if constexpr (RM) {
        // base and +-1 sum apart: 4 .. 7 hand theirs to 0 .. 3, whose sums are added in order; the scale multiplies the finished one
        const int mine = (wave & 3) * 2 * kSet;
        if (wave >= 4) {
            put(mine, [&](int r, int ct) { return acc[r][ct]; });
            put(mine + kSet, [&](int r, int ct) { return dsum[r][ct]; });
        }
        __syncthreads();
        if (wave < 4) {
            put(mine, [&](int r, int ct) { return acc[r][ct] + *(const float4v*)(smem + mine + lane_at + (r * MT + ct) * 1024); });
            put(mine + kSet, [&](int r, int ct) { return dsum[r][ct] + *(const float4v*)(smem + mine + kSet + lane_at + (r * MT + ct) * 1024); });
        }
        __syncthreads();
        write_y(0, 1, true);
    } else {
        // as the decode kernel: every wavefront scales its own part, and the parts are added in order
        bool any_inf = false;
#pragma unroll
        for (int ct = 0; ct < MT; ++ct) any_inf = any_inf || __builtin_isinf(scale_of(ct));
        any_inf = any_inf && !a.inf_in_parts;
        auto scaled = [&](int r, int ct) {
            const float al = scale_of(ct);
            float4v p = acc[r][ct];
            if (!any_inf || !__builtin_isinf(al)) {
#pragma unroll
                for (int e = 0; e < 4; ++e) p[e] = acc[r][ct][e] + al * dsum[r][ct][e];
            }
            return p;
        };
        if (!any_inf) {
            put(wave * kSet, scaled);
            __syncthreads();
            write_y(0, subs, false);
            return;
        }
        // An infinite scale would make NaN of a part that is zero: it multiplies the finished sum, which goes behind the parts.
        for (int s = 0; s < subs; ++s) {
            if (sub == s) put(wave * kSet, [&](int r, int ct) { return dsum[r][ct]; });
            __syncthreads();
            for (int idx = threadIdx.x; idx < R * MT * 256; idx += kWideWaves * kWave) {
                float t = 0.f;
                for (int w = 0; w < nw; ++w) t += *(const float*)(smem + (w * subs + s) * kSet + idx * 4);
                *(float*)(smem + 8 * kSet + idx * 4) = t;
            }
            __syncthreads();
            if (sub == s) put(wave * kSet, scaled);
            __syncthreads();
            write_y(s, 1, true);
            __syncthreads();
        }
    }
}

template <int R, int MT, bool RM, bool TILE_SUMS>
static hipError_t launch_wide_inst(const WideArgs& args, hipStream_t st) {
    auto kernel = linear_wide_kernel<R, MT, RM, TILE_SUMS>;
    constexpr int lds = WideLds<R, MT>::kTotal;
    static_assert(lds <= 160 * 1024, "LDS budget");
    static PerDeviceOnce once;
    const hipError_t ea = once.run([&] {
        hipFuncAttributes fa;
        const hipError_t e = hipFuncGetAttributes(&fa, (const void*)kernel);
        if (e != hipSuccess) return e;
        if (fa.sharedSizeBytes != 0) return hipErrorInvalidValue;   // the table must start at LDS address 0
        return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    });
    if (ea != hipSuccess) return ea;
    const int per_group = R * (RM ? 1 : kWideWaves / wide_k_waves(args.KT));
    const unsigned groups = (unsigned)((args.row_blocks + per_group - 1) / per_group);
    const unsigned chunks = (unsigned)((args.n_tiles + args.tiles_per_chunk - 1) / args.tiles_per_chunk);
    hipLaunchKernelGGL(kernel, dim3((groups + 7) / 8 * 8 * chunks), dim3(kWideWaves * kWave), lds, st, args);
    return hipGetLastError();
}

// args.n_tiles column tiles (1 .. kWideMaxTiles) in chunks of args.tiles_per_chunk (1 .. kWideMaxChunk), R row blocks per workgroup
hipError_t launch_linear_wide(const WideArgs& args, int R, bool rowmajor, hipStream_t st) {
    if (args.n_tiles < 1 || args.n_tiles > kWideMaxTiles || args.tiles_per_chunk < 1 || args.in < 128 ||
        args.in % kWideUnit != 0 || args.units != args.in / kWideUnit || args.out < 1 || (R != 1 && R != 2) ||
        (rowmajor && !args.packed_by_tenant))
        return hipErrorInvalidValue;
    const int n = args.tiles_per_chunk;
    if (n < 1 || n > wide_max_chunk(R, args.KT, rowmajor)) return hipErrorInvalidValue;
    // tiled: the +-1 sums of k tiles are added up apart, unless no wavefront has more than one
    auto go = [&](auto r_tag, auto mt_tag) {
        constexpr int RR = decltype(r_tag)::value, M = decltype(mt_tag)::value;
        if (rowmajor) return launch_wide_inst<RR, M, true, false>(args, st);
        if constexpr (RR == 2 && M == 6) return launch_wide_inst<RR, M, false, false>(args, st);
        else return launch_wide_inst<RR, M, false, true>(args, st);
    };
    auto go_r = [&](auto r_tag) {
        if (n <= 2) return go(r_tag, std::integral_constant<int, 2>{});
        if (n <= 4) return go(r_tag, std::integral_constant<int, 4>{});
        if (n <= 6) return go(r_tag, std::integral_constant<int, 6>{});
        if constexpr (decltype(r_tag)::value == 1) {
            if (n <= 8) return go(r_tag, std::integral_constant<int, 8>{});
            return go(r_tag, std::integral_constant<int, 10>{});
        }
        return hipErrorInvalidValue;
    };
    return R == 1 ? go_r(std::integral_constant<int, 1>{}) : go_r(std::integral_constant<int, 2>{});
}

}  // namespace bd

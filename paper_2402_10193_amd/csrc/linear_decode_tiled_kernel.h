// Decode kernel of the multi-tenant linear (Eq. 6 of the paper) over the tiled serving layout:
//     y[t, n] = sum_k x[t,k] W_base[n,k]  +  alpha_e * sum_k x[t,k] s_e[n,k],   e = tenant(t).
//
// At decode every token has its own tenant, so a packed sign word is used exactly once and
// the kernel is a pure stream: per byte of base weight it must turn B/16 sign bits into
// multiply-add operands.  Both products run on v_mfma_f32_16x16x32_f16 (A = 16 output rows x
// 32 k, B = 32 k x 16 token columns, tokens sorted by tenant); a delta "job" is one tenant's
// signs against all 16 columns, of which only that tenant's columns are kept.
//
// Sign expansion.  A byte of 8 signs becomes the 8 fp16 values +-1.0 (one 128-bit MFMA operand
// register group) by ONE look-up in LDS: the table has 256 entries x 16 B, replicated 16 times
// so that lane l reads copy l % 16 and a group of 16 lanes never shares a bank.  The address
// is built by one v_perm_b32 (sign byte -> address bits 8..15, lane copy -> bits 4..7), so the
// vector ALU spends one instruction per 8 signs; the LDS read port does the rest, next to the
// matrix pipe.  (Expanding with and-or instructions costs >= 8 per 8 signs and, at one token per
// tenant, makes the vector ALU the bottleneck long before HBM.)
//
// Decomposition.  The grid is persistent: one workgroup per compute unit, each owning a
// contiguous range of the launch's 16-row blocks (all matrices of a grouped launch laid end to
// end); its wavefronts split the k tiles into contiguous ranges.  A task = one (row block, k tile):
// 8 KiB of base (8 loads of 1 KiB), 512 B of signs per job (one 64-bit load per lane) and the
// 16 x 256 block of x, which each lane loads straight from global memory (L2 hits) in B-operand
// order: no staging, no barrier in the loop.  When a wavefront has at most two k tiles its x
// stays in registers for all of its row blocks (x is then fetched once per workgroup instead
// of once per task; the L1 is an in-order queue, so every x request it does not carry leaves
// room for a weight request).  Otherwise x is double-buffered per task.
// Everything of task t+1 is requested while task t is being multiplied: W[v] right after its
// MFMA, the signs of job j right after their addresses are formed.  Per row block the
// wavefronts' partial tiles go to LDS slots and are added in a fixed order when the slots are
// full or the work is done; y is written once.
//
// Quantised base (Q8; Sec. 4.2 of the paper, quantized base models).  The base tile then holds one
// byte per weight, u = q + 128, and a lane's 8 bytes of a slice become the MFMA operand by four
// v_perm_b32: byte u next to the constant 0x64 is the fp16 number 1024 + u, exactly.  The base
// accumulator therefore holds sum_k x (1152 + q); a second MFMA per slice with an all-ones A operand
// accumulates sum_k x, and the finished row block is scale[n] * (acc - 1152 * sum_k x): no
// arithmetic per weight beyond the byte shuffle.
//
// Row-major tensors (RM; what bd_compress writes and bd_linear_multitenant takes).  The same kernel reads W
// [out, in] fp16 and packed signs [out, in/32] as they are: slice v of a base tile is then 16 rows x 64 bytes
// (fetched with 16 lanes side by side in a row and turned into operand order through LDS rows of the wavefront's own), and a
// tenant's signs of a tile are 16 rows x 32 bytes: lane (r, j) fetches those of row r for job slot 4 p + j, and the lanes of
// a row exchange them so that lane (r, g) holds byte g of all eight words for all four slots (byte shuffles inside the lane,
// v_permlane32_swap / v_permlane16_swap between them: six vector instructions per job and task).  The tenants' pointers
// come from the caller's device table instead of the kernel arguments.  Long rows with many slots: see S4.
//
// This header is the kernel; linear_decode_tiled.hip, linear_decode_tiled_q8.hip and linear_decode_rowmajor.hip
// instantiate it for the fp16 base, the 8-bit base and the row-major tensors (three translation units, so that
// they compile side by side).
#pragma once

#include <type_traits>

#include "bd_device.h"
#include "bd_launch.h"
#include "bd_tiled.h"

namespace bd {

namespace {

constexpr int kLutBytes = 256 * 16 * 16;          // 256 entries x 16 copies x 16 B
constexpr int kRedBytesPerWave = 16 * 16 * 4;     // one 16 x 16 fp32 tile
constexpr int kMaxWavesTiled = 8;
// x staging of one wavefront: 16 token rows x (512 B + 16 B pad), the pad spreads the 16 rows over all banks
constexpr int kStageRowBytes = kTileK * 2 + 16;
constexpr int kStageBytes = 16 * kStageRowBytes;
// LDS after the table: one region per wavefront = slots for the partial tiles of finished row blocks.
// Resident x is staged there before the first task (the slots overlay the staging rows).
// Row-major fp16 base: behind the slots a room of 16 rows x 256 bytes, in which half a base tile at a time goes from rows
// to operand order.
constexpr int kRoomBytes = 16 * 256;
template <int XSTEPS, bool ROOM> struct LdsPlan {
    static constexpr int kRedSlots = ROOM ? 4 : 8;   // 16 x 16 tiles; a row block takes one per column tile
    static constexpr int kRoom = kRedSlots * kRedBytesPerWave;   // where the room starts in the region
    static constexpr int kUsed = kRoom + (ROOM ? kRoomBytes : 0);
    static constexpr int kRegion = (XSTEPS > 0 && kStageBytes > kUsed) ? kStageBytes : kUsed;
    // behind the regions: (span, token) of every column of both column tiles, for the threads that write y
    static constexpr int kMeta = kLutBytes + kMaxWavesTiled * kRegion;
    // row-major: the address of every job slot's signs
    static constexpr int kPtr = kMeta + kTiledMaxCt * kTiledMaxTokens * 8;
    static constexpr int kTotal = kPtr + kTiledMaxCt * kTiledMaxJobs * 8;
};
static_assert(LdsPlan<0, false>::kTotal <= 160 * 1024 && LdsPlan<2, false>::kTotal <= 160 * 1024 && LdsPlan<0, true>::kTotal <= 160 * 1024 &&
                  LdsPlan<2, true>::kTotal <= 160 * 1024,
              "LDS budget");

__device__ __forceinline__ void lds_wave_sync() {   // order this wavefront's LDS writes before its later reads
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Streamed x through a buffer resource: this offset is its end, where a load gives zeros without a memory access.  (x has fewer than
// 2^32 bytes, rows of whole 64 bytes: the host checks it, so that no slice of a row begins this far.)
constexpr uint32_t kXNowhere = 0xFFFFFFF0u;
typedef const void __attribute__((address_space(1)))* gptr_t;
typedef const u32x4 __attribute__((address_space(3)))* lds_u32x4_ptr;

__device__ __forceinline__ u32x4 ldg16_stream(const unsigned char* base, uint32_t off) {
    return __builtin_nontemporal_load((const u32x4*)(base + off));
}
__device__ __forceinline__ u32x2 ldg8_stream(const unsigned char* base, uint32_t off) {
    return __builtin_nontemporal_load((const u32x2*)(base + off));
}
__device__ __forceinline__ u32x4 ldg16(const unsigned char* base, uint32_t off) {
    return *(const u32x4*)(base + off);
}

// The MFMA operand of slice v of a job's tile: byte v of the lane's sign words -> table entry.
// `lanebits` = 16 * (lane % 16) in byte 0; the selector puts sign byte (v % 4) of word v / 4
// into byte 1 and zeros above: address = 256 * byte + 16 * copy (the table starts at LDS address 0).
__device__ __forceinline__ u32x4 lut_read(const u32x2 s, const int v, const uint32_t lanebits) {
    const uint32_t addr = __builtin_amdgcn_perm(s[v >> 2], lanebits, 0x0C0C0000u | ((4u + (v & 3)) << 8));
    return *(lds_u32x4_ptr)(uintptr_t)addr;
}

// Row-major signs, four job slots at a time.  In: lane (r, j) = (lane % 16, lane / 16) holds the 8 words that row r of job slot j
// has for the tile; byte i of word w is the sign byte of slice w for lane group i.  Out: s[j] = byte g of words 0..3 and of
// words 4..7 of job slot j, in lane (r, g): what the tiled layout holds there.
__device__ __forceinline__ void rm_turn_signs(const u32x4 lo, const u32x4 hi, u32x2 (&s)[4]) {
    const u32x4 a = turn_sign_words(lo), b = turn_sign_words(hi);
#pragma unroll
    for (int j = 0; j < 4; ++j) s[j] = u32x2{a[j], b[j]};
}
// Row-major signs, one job slot at a time (see S4).  In: this lane's words 2 g and 2 g + 1 of its row (lane (r, g) = (lane % 16, lane / 16)); byte i of
// word w is the sign byte of slice w for lane group i.  Out: s[0] = byte g of words 0, 1, 4, 5 and s[1] = byte g of
// words 2, 3, 6, 7 (in that order), i.e. everything lane (r, g) needs.  All 64 lanes must be active.
__device__ __forceinline__ u32x2 rm_gather_sign_bytes(const u32x2 w) {
    // bytes for lane groups 0, 1 and for 2, 3, the two words interleaved
    const uint32_t p = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);
    const uint32_t q = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);
    // lanes 32..63 of p against lanes 0..31 of q: groups 0, 1 now hold both halves' p, groups 2, 3 both halves' q
    const auto h = __builtin_amdgcn_permlane32_swap(p, q, false, false);
    // split by the parity of the byte index, then trade with the neighbouring group
    const uint32_t u = __builtin_amdgcn_perm(h[1], h[0], 0x05040100u);
    const uint32_t t = __builtin_amdgcn_perm(h[1], h[0], 0x07060302u);
    const auto f = __builtin_amdgcn_permlane16_swap(u, t, false, false);
    return u32x2{f[0], f[1]};
}
// Row-major 8-bit base.  In: the 16 bytes lane (r, g) loaded, q[row r][64 i + 16 g ..] (two's complement).  Out: the
// lane's 8 bytes of slice 2 i in words 0, 1 and of slice 2 i + 1 in words 2, 3, as u = q + 128 (what the tiled 8-bit base
// holds).  The four lanes of a row hold [lo, hi] halves; lane g' needs half g' % 2 of lane g' / 2 (slice 2 i) and of
// lane 2 + g' / 2 (slice 2 i + 1): a swap between neighbouring rows of 16 lanes, then one between the wavefront's halves.
__device__ __forceinline__ u32x4 rm_gather_q8(const u32x4 w) {
    u32x4 r;
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const auto s16 = __builtin_amdgcn_permlane16_swap(w[d], w[2 + d], false, false);
        const auto s32 = __builtin_amdgcn_permlane32_swap(s16[0], s16[1], false, false);
        r[d] = s32[0] ^ 0x80808080u;
        r[2 + d] = s32[1] ^ 0x80808080u;
    }
    return r;
}
// slice v of the gathered bytes: word (v / 2) % 2, byte v % 2 + 2 * (v / 4)
__device__ __forceinline__ u32x4 lut_read_rm(const u32x2 s, const int v, const uint32_t lanebits) {
    const uint32_t addr = __builtin_amdgcn_perm(s[(v >> 1) & 1], lanebits, 0x0C0C0000u | ((4u + ((v & 1) | ((v & 4) >> 1))) << 8));
    return *(lds_u32x4_ptr)(uintptr_t)addr;
}

}  // namespace

// XSTEPS = 1 or 2: every wavefront has exactly that many k tiles and keeps their x in registers.
// XSTEPS = 0: any number of k tiles per wavefront, x double-buffered per task.
// NCT = 2 (streamed x only): 17..32 tokens as two column tiles; the tasks of one (row block, k tile)
// then come in pairs that share the base registers, so the base is still read once.
// RM: row-major W (fp16, or the int8 q of the 8-bit base with its `out` scales) and packed signs (one matrix,
// in % 128 == 0) instead of the tiled tensors.
// (The row-major fp16 base passes through LDS rows unless x of two k tiles and the signs of more than 12 slots leave no
// registers for it; streaming x instead costs more: 11008 x 4096 with 16 tenants 49 against 57 us.)
constexpr bool rm_base_through_lds(int nj, int xsteps, bool q8, bool rm) { return rm && !q8 && !(xsteps == 2 && nj > 12); }
// RG = 2 (streamed x): a wavefront works on two row blocks of a matrix at the same time (k tile by k tile, one after the other), so that x of a
// k tile is fetched once for both: it comes from L2, but its lines take their places among the pending requests of the L1, which are what
// limits the stream (32 tokens: 16 KiB of x next to 8 KiB of base and 16 of signs per task).  The sums of the row block that is not being
// multiplied change places with the other's: 16 moves per column tile and task.  Without any fetch of x a 70B layer with 32 tokens
// took 877 us where it took 1064.  launch_nj has the line between one row block and two.
// S4 (row-major): the signs are fetched for four job slots at a time, 16 bytes per lane, every lane a row of a slot (128 cycles of
// the address unit for four slots), instead of 8 bytes per lane, four lanes a row, slot by slot (256 cycles).  But a row's 32
// bytes then come in two requests: launch_nj has the line between the two.
template <int NJ, int XSTEPS, int NCT, bool Q8, bool RM = false, bool S4 = RM, int RG = 1>
__global__ __launch_bounds__(kMaxWavesTiled * kWave) void linear_decode_tiled_kernel(const TiledArgs a) {
    constexpr uint32_t kWTile = Q8 ? kTileBaseQ8Bytes : kTileBaseBytes;   // bytes of one base tile
    constexpr int kWLoads = Q8 ? 4 : 8;                                   // 1 KiB loads per base tile
    extern __shared__ __align__(16) unsigned char smem[];   // [0, 64 KiB): table; then one region per wavefront
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int nw = blockDim.x >> 6;
    const int c = lane & 15;   // A row (output row) for loads, B/D column (token) for MFMA operands and results
    const int g = lane >> 4;
    constexpr bool ROOM = rm_base_through_lds(NJ, XSTEPS, Q8, RM);
    using Plan = LdsPlan<XSTEPS, ROOM>;
    static_assert((NCT == 1 && RG == 1) || XSTEPS == 0, "two column tiles and two row blocks only with streamed x");
    static_assert(RG == 1 || RG == 2, "the other row block's sums change places with this one's");
    // Touch every 64-byte line of the kernel arguments at once: the first read of a line is a trip
    // to memory, and taken one after the other (pointer tables are indexed by values read before)
    // those trips would delay the first weight request by microseconds.
    {
        const unsigned char __attribute__((address_space(4)))* ka =
            (const unsigned char __attribute__((address_space(4)))*)__builtin_amdgcn_kernarg_segment_ptr();
        constexpr int kLines = (int)((sizeof(TiledArgs) + 63) / 64);
        uint32_t touched[kLines];
#pragma unroll
        for (int i = 0; i < kLines; ++i) {
            const uint32_t off = (uint32_t)i * 64u;
            asm volatile("s_load_dword %0, %1, %2" : "=s"(touched[i]) : "s"(ka), "s"(off));
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < kLines; ++i) asm volatile("" ::"s"(touched[i]));
    }
    const int KT = a.KT;
    const int rb_total = a.rb_end[a.n_mats - 1];
    // this workgroup's row blocks [r0, r1) of the concatenated matrices (the host keeps grid <= rb_total)
    const int r0 = (int)((int64_t)blockIdx.x * rb_total / gridDim.x);
    const int r1 = (int)((int64_t)(blockIdx.x + 1) * rb_total / gridDim.x);
    const int n_rb = r1 - r0;
    // This wavefront's k tiles: kb, kb + kstride, ... (`steps` of them).  Tiled tensors: a contiguous range.  Row-major: every
    // nw-th tile, so that the wavefronts of a workgroup are on neighbouring tiles at the same time: a 128-byte line of a
    // row's signs covers four k tiles, and taken by one wavefront in four consecutive tasks it would come from HBM four times.
    const int kb = RM ? wave : wave * KT / nw;
    const int kstride = RM ? nw : 1;
    const int steps = XSTEPS > 0 ? XSTEPS : (RM ? (KT - wave + nw - 1) / nw : (wave + 1) * KT / nw - kb);
    const bool have_work = n_rb > 0 && steps > 0;

    auto mat_of = [&](const int rbg, int& m, int& rb) {
        m = 0;
        if (a.n_mats > 1 && rbg >= a.rb_end[0]) m = 1;
        if (a.n_mats > 2 && rbg >= a.rb_end[1]) m = 2;
        rb = rbg - (m > 0 ? a.rb_end[m - 1] : 0);
    };

    // ---- pointers of the matrix whose tiles are being REQUESTED (the task being multiplied only
    // needs registers); reloaded from the kernel arguments when the requests cross into the next matrix
    int m_req, rb_req;
    mat_of(r0, m_req, rb_req);
    const unsigned char* wt = (const unsigned char*)a.wt[m_req];
    const unsigned char* sp[NCT][NJ];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
        for (int j = 0; j < NJ; ++j) sp[ct][j] = RM ? nullptr : (const unsigned char*)a.signs[ct][m_req][j];
    // Row-major: the tenants' pointers come from the caller's table in device memory and wait in LDS; a lane takes the one of
    // the job slot it fetches for.
    if constexpr (S4) {
        if (threadIdx.x < kTiledMaxCt * kTiledMaxJobs)
            *(uint64_t*)(smem + Plan::kPtr + threadIdx.x * 8) =
                (uint64_t)a.packed_by_tenant[a.job_tenant[threadIdx.x / kTiledMaxJobs][threadIdx.x % kTiledMaxJobs]];
    }
    // One slot at a time: sixteen pointers held as
    // scalars cannot be dropped and fetched again like kernel arguments, and would push the kernel's vector
    // registers into scratch; so lane j of one register pair holds the pointer of job slot j, and a sign load
    // takes its base address from there with two v_readlane.
    uint32_t ptr_lo[NCT], ptr_hi[NCT];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
        ptr_lo[ct] = ptr_hi[ct] = 0u;
        if constexpr (RM && !S4) {
            int tenant_l = a.job_tenant[ct][0];
#pragma unroll
            for (int i = 1; i < kTiledMaxJobs; ++i) tenant_l = (lane == i) ? a.job_tenant[ct][i] : tenant_l;
            const uint64_t pv = (uint64_t)a.packed_by_tenant[tenant_l];
            ptr_lo[ct] = (uint32_t)pv;
            ptr_hi[ct] = (uint32_t)(pv >> 32);
        }
    }
    auto sign_ptr = [&](const int ct, const int j) -> const unsigned char* {
        if constexpr (RM) {
            const uint32_t lo = __builtin_amdgcn_readlane(ptr_lo[ct], j), hi = __builtin_amdgcn_readlane(ptr_hi[ct], j);
            return (const unsigned char*)(((uint64_t)hi << 32) | lo);
        } else {
            return sp[ct][j];
        }
    };
    // Byte offsets of a task's loads = a uniform part (tile) + this lane's part.  Tiled: the lane's part is its place
    // inside a tile.  Row-major: the uniform part is the k tile only and the lane's part carries the row, so it
    // changes with the row block (rows beyond `out` read the last row again; their results are never stored).  A row-major
    // fp16 base is fetched with 16 lanes side by side in a row: load 4 h + j covers rows 4 j .. 4 j + 3 of half h of the tile,
    // 16-byte chunk c ^ row in lane c of the row, and is turned into operand order in the wavefront's room of LDS.  (In
    // operand order neighbouring lanes are on different rows, every lane an access of its own: 64 cycles of the address
    // unit per load, 512 per task, and with the signs twice what the memory leaves time for.)
    uint32_t wrow[4] = {0u, 0u, 0u, 0u};
    uint32_t lane16 = (uint32_t)lane * 16u, lane8 = (uint32_t)lane * 8u;
    auto rm_lane_offsets = [&](const int rb) {
        const int row = min(rb * kTileRows + c, a.out[0] - 1);
        lane16 = (uint32_t)row * ((uint32_t)a.in * (Q8 ? 1u : 2u)) + (uint32_t)g * 16u;
        lane8 = (uint32_t)row * ((uint32_t)a.in >> 3) + (S4 ? 0u : (uint32_t)g * 8u);
        if constexpr (ROOM) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                wrow[j] = (uint32_t)min(rb * kTileRows + 4 * j + g, a.out[0] - 1) * ((uint32_t)a.in * 2u) + ((uint32_t)(c ^ (4 * j + g)) << 4);
        }
    };
    if constexpr (RM) rm_lane_offsets(rb_req);
    auto w_off = [&](const int rb, const int kt) {   // uniform byte offset of tile (rb, kt) of the base
        return RM ? (uint32_t)kt * (uint32_t)(kTileK * (Q8 ? 1 : 2)) : (uint32_t)(rb * KT + kt) * kWTile;
    };
    auto s_off = [&](const int rb, const int kt) {   // ... of a tenant's signs
        return RM ? (uint32_t)kt * (uint32_t)(kTileK / 8) : (uint32_t)(rb * KT + kt) * (uint32_t)kTileSignBytes;
    };
    constexpr uint32_t kSliceStride = RM ? 64u : 1024u;   // bytes between a lane's loads of consecutive slices
    // The tiled tensors are read once, whole cache lines at a time, with non-temporal loads (nothing of a line is
    // needed again).  Row-major, a load takes half a line of the base and a quarter of a line of signs per row; the rest
    // of the line belongs to the next slice or to the neighbouring wavefront's tiles, so those loads are ordinary ones
    // and the line stays in L2 for them (non-temporal, every line came from HBM 1.6 to 2.3 times).
    auto ld_w = [](const unsigned char* p, const uint32_t off) { return RM ? ldg16(p, off) : ldg16_stream(p, off); };
    auto ld_s = [](const unsigned char* p, const uint32_t off) {
        return RM ? *(const u32x2*)(p + off) : ldg8_stream(p, off);
    };
    // Row-major, `in` = 128 mod 256: the last k tile of a row has 4 slices.  No load may reach beyond the row (the
    // last row ends the tensor), so slices 4..7 of such a tile read slices 0..3 again and are replaced by zeros when
    // they are multiplied; words 4..7 of its signs are words 0..3 again (any valid words do: their x is zero).  All of it is
    // uniform arithmetic per task, no branch around a load.
    const int kt_short = (RM && (a.in % kTileK) != 0) ? KT - 1 : -1;
    auto w_base_hi = [&](const int kt) {   // the pointer slices 4..7 of tile kt are read through
        return (RM && kt == kt_short) ? wt - (kWLoads / 2) * kSliceStride : wt;
    };
    // request number v of a base tile (woff: the tile's offset, the lane's part included unless ROOM)
    auto ld_base = [&](const unsigned char* const hi, const uint32_t woff, const int v) __attribute__((always_inline)) {
        const unsigned char* const p = v >= kWLoads / 2 ? hi : wt;
        if constexpr (ROOM) {
            uint32_t r = wrow[v & 3];
            asm volatile("" : "+v"(r));
            return ldg16(p, woff + r + (v >= 4 ? 256u : 0u));
        } else {
            return ld_w(p, woff + (uint32_t)v * kSliceStride);
        }
    };
    // Row-major signs of four job slots 4 p .. 4 p + 3: lane (c, j) the 32 bytes that row c of slot 4 p + j has for the tile.
    typedef const u32x4 __attribute__((address_space(1)))* global_u32x4;
    auto ld_s4 = [&](u32x2 (&s4)[4], const int ct, const int p, const int kt) __attribute__((always_inline)) {
        uint32_t l8 = lane8;
        asm volatile("" : "+v"(l8));
        const uint64_t ptr = *(const uint64_t*)(smem + Plan::kPtr + (ct * kTiledMaxJobs + 4 * p + g) * 8) + l8 + (uint32_t)kt * (uint32_t)(kTileK / 8);
        const u32x4 lo = *(global_u32x4)ptr, hi = *(global_u32x4)(ptr + (kt == kt_short ? 0u : 16u));
        s4[0] = u32x2{lo[0], lo[1]};
        s4[1] = u32x2{lo[2], lo[3]};
        s4[2] = u32x2{hi[0], hi[1]};
        s4[3] = u32x2{hi[2], hi[3]};
    };
    auto turn_s4 = [&](u32x2 (&s4)[4]) __attribute__((always_inline)) {
        rm_turn_signs(u32x4{s4[0][0], s4[0][1], s4[1][0], s4[1][1]}, u32x4{s4[2][0], s4[2][1], s4[3][0], s4[3][1]}, s4);
    };

    // one slot at a time: in a short last tile lane groups 2, 3 read the row's first sign words (any valid words do)
    auto s_lane_off = [&](const uint32_t off_u, const uint32_t l8, const int kt) {
        uint32_t off = off_u + l8;
        if constexpr (RM) off = (kt == kt_short && g >= 2) ? l8 - (uint32_t)g * 8u : off;
        return off;
    };

    // x of one k tile is a [16 tokens][256] fp16 block.  It is fetched with loads whose lanes are
    // contiguous in memory (load i: token rows 2i and 2i+1, 512 B each) and brought into B-operand
    // order (lane (c, g): row c, elements 32 v + 8 g ..) through this wavefront's LDS staging rows:
    // fetching it in operand order directly would make every lane its own 16-byte access.
    // Rows of columns beyond T read token col_token[0] (valid memory); their results are never stored.
    const unsigned char* xg = (const unsigned char*)a.x;
    const int xh = lane >> 5;                                   // which of the two rows of a load
    const uint32_t xcol = (uint32_t)(lane & 31) * 16u;          // byte inside the tile row
    const int k_ragged = (a.in % kTileK != 0) ? KT - 1 : -1;    // the tile that reaches beyond `in`, if any
    const uint32_t row_bytes = (uint32_t)a.in * 2u;
    auto x_fetch = [&](u32x4 (&xraw)[8], const int kt) {
        uint32_t xc = xcol;
        asm volatile("" : "+v"(xc));   // keep "base + lane offset" a 32-bit offset (see task())
        const uint32_t off = xc + (uint32_t)kt * (uint32_t)(kTileK * 2);
        const bool inside = (kt != k_ragged) || (kt * kTileK + (lane & 31) * 8 < a.in);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int ra = 2 * i < a.T[0] ? a.col_token[0][2 * i] : a.col_token[0][0];
            const int rbw = 2 * i + 1 < a.T[0] ? a.col_token[0][2 * i + 1] : a.col_token[0][0];
            const uint32_t tokoff = (uint32_t)(xh ? rbw : ra) * row_bytes;
            xraw[i] = u32x4{0u, 0u, 0u, 0u};
            if (inside) xraw[i] = ldg16(xg, tokoff + off);
        }
    };
    // Streamed x (a fresh tile per task) is fetched in operand order directly: lane (c, g), slice v reads
    // x[token of column c][256 kt + 32 v + 8 g ..]; a trip through LDS per task would sit on the critical path.
    uint32_t xlane[NCT];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
        int tok_c = a.col_token[ct][0];
#pragma unroll
        for (int i = 0; i < kTiledMaxTokens; ++i) tok_c = (c == i && i < a.T[ct]) ? a.col_token[ct][i] : tok_c;
        xlane[ct] = (uint32_t)tok_c * row_bytes + (uint32_t)g * 16u;
    }
    // A slice that lies beyond `in` (ragged tile only) is asked for at the end of the buffer resource and arrives as zeros: every path
    // issues the same eight loads, so that the count of loads in flight at any later point is known at compile time and nothing
    // has to wait for more than it needs, and no register is written again behind the load.
    const auto xrsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, kXNowhere, 0x00020000);
    auto x_fetch_operands = [&](u32x4 (&xop)[8], const int kt, const int ct) __attribute__((always_inline)) {
        uint32_t xl = ct == 0 ? xlane[0] : xlane[NCT - 1];
        asm volatile("" : "+v"(xl));
        const uint32_t off = xl + (uint32_t)kt * (uint32_t)(kTileK * 2);
        const int n_in = (a.in - kt * kTileK - 8 * g + 31) >> 5;   // this lane's slices inside the row (may be negative)
#pragma unroll
        for (int v = 0; v < 8; ++v) xop[v] = __builtin_amdgcn_raw_buffer_load_b128(xrsrc, v < n_in ? off + v * 64 : kXNowhere, 0, 0);
    };
    // ---- requests of the first task: x first, then the base, (the table,) then the signs.  x is small and every
    // workgroup asks for the same lines; asked for behind the first base tiles of all compute units (16 MB) it arrives
    // microseconds after them and the first base product waits for it.  (Measured: 1.3 % on launches of one matrix, nothing
    // on the grouped launches, whose end is set by the stream.)
    constexpr int XR = XSTEPS > 0 ? XSTEPS : NCT;   // x register sets in operand order
    u32x4 xs[XR][8];
    u32x4 xraw[XR][8];                            // resident x as fetched; streamed x, one column tile: the next k tile's operands
    if (have_work) {
        if constexpr (XSTEPS > 0) x_fetch(xraw[0], kb);
        else {
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct) x_fetch_operands(xs[XSTEPS > 0 ? 0 : ct], kb, ct);
        }
        if constexpr (XSTEPS == 2) x_fetch(xraw[1], kb + kstride);
    }
    u32x4 wr[kWLoads];   // fp16 base: slice v; 8-bit base: slices 2 i and 2 i + 1 (8 bytes each)
    constexpr int kSg = (NJ + 3) / 4;
    u32x2 sr[kSg][4];    // job slot j: sr[j / 4][j % 4] (row-major: four slots' words as fetched until the first of them is due)
    if (have_work) {
        const uint32_t woff0 = w_off(rb_req, kb) + (ROOM ? 0u : lane16);
        const unsigned char* const wt_hi0 = w_base_hi(kb);
#pragma unroll
        for (int v = 0; v < kWLoads; ++v) wr[v] = ld_base(wt_hi0, woff0, v);
    }

    // ---- the table: entry b, copy cp at 256 b + 16 cp; element e = bit e of b ? +1.0 : -1.0.
    // Built (and the workgroup synchronised) while only the first base requests are in flight: the
    // later requests queue up behind the memory system, and a barrier behind them would hold the
    // first multiplications back by microseconds.
    // Consecutive lanes write consecutive 16-byte copies (16 per entry), a wavefront 1 KiB at a stretch: with a
    // lane per entry the writes of a wavefront were 128 bytes apart, eight of them on every bank.
    // Entry b = 32 i + 4 j + lane / 16: eight writes (j) per turn of the loop, whose words are constants but for bits 0 and 1 (the lane's) and
    // 5 to 7 (the turn's).  With its words formed for every write on its own, the loop was 27 instructions per KiB, turned 64 times by a single wavefront and
    // 32 times by two, and the time of a short launch hung on where the compiler had placed it: 2048 x 512, two wavefronts, 1 tenant 6.4 us,
    // but 7.3 where it began 28 bytes behind a multiple of 32 (in kernels of 2, 4 and 8 job slots); now 4.9, 2048 x 256 8.9 -> 5.6, 2048 x 1024 5.7 -> 5.3.
    {
        const uint32_t e0 = 0xBC00BC00u ^ ((uint32_t)(g & 1) << 15) ^ ((uint32_t)(g >> 1) << 31);
        for (int i = wave; i < 8; i += nw) {
            unsigned char* const at = smem + i * 8192 + lane * 16;
            const uint32_t e3 = 0xBC00BC00u ^ (((uint32_t)i >> 1 & 1u) << 15) ^ (((uint32_t)i >> 2) << 31);
#pragma unroll
            for (uint32_t j = 0; j < 8; ++j)
                *(u32x4*)(at + j * 1024) = u32x4{e0, 0xBC00BC00u ^ ((j & 1u) << 15) ^ ((j >> 1 & 1u) << 31),
                                                 0xBC00BC00u ^ ((j >> 2) << 15) ^ (((uint32_t)i & 1u) << 31), e3};
        }
    }
    // What the write of y needs per column, read from the kernel arguments with a lane's own index (a load from memory)
    // here, where it waits with everything else, and from LDS when a row block is finished: at the end of a launch a trip
    // to memory for it would be added to the launch's time.
    if (threadIdx.x < kTiledMaxCt * kTiledMaxTokens) {
        const int ct = threadIdx.x / kTiledMaxTokens, col = threadIdx.x % kTiledMaxTokens;
        *(u32x2*)(smem + Plan::kMeta + threadIdx.x * 8) = u32x2{(uint32_t)a.col_span[ct][col], (uint32_t)a.col_token[ct][col]};
    }
    __syncthreads();


    unsigned char* const region = smem + kLutBytes + wave * Plan::kRegion;
    auto x_to_operands = [&](const u32x4 (&xraw)[8], u32x4 (&xop)[8]) {
        lds_wave_sync();   // earlier reads of the staging rows are done
#pragma unroll
        for (int i = 0; i < 8; ++i) *(u32x4*)(region + (2 * i + xh) * kStageRowBytes + xcol) = xraw[i];
        lds_wave_sync();
#pragma unroll
        for (int v = 0; v < 8; ++v) xop[v] = *(const u32x4*)(region + c * kStageRowBytes + 64 * v + 16 * g);
    };

    // a row-major base tile, as fetched -> operands, in place
    auto w_turn = [&]() __attribute__((always_inline)) {
        unsigned char* const room = region + Plan::kRoom;
        const uint32_t get = (uint32_t)c * 256u + ((uint32_t)(c ^ g) << 4);   // chunk 4 v + g of row c is at get ^ 64 v
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            lds_wave_sync();
#pragma unroll
            for (int j = 0; j < 4; ++j) *(u32x4*)(room + j * 1024 + lane * 16) = wr[4 * h + j];
            lds_wave_sync();
#pragma unroll
            for (int v = 0; v < 4; ++v) wr[4 * h + v] = *(const u32x4*)(room + (get ^ (64u * v)));
        }
    };

    if (have_work) {
        // (row-major: resident x, requested first, takes its registers before the signs are requested; all three at once do
        // not fit)
        if constexpr (ROOM) {
#pragma unroll
            for (int i = 0; i < (XSTEPS > 0 ? XR : 0); ++i) x_to_operands(xraw[i], xs[i]);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (S4) {
#pragma unroll
            for (int p = 0; p < kSg; ++p) ld_s4(sr[p], 0, p, kb);
        } else {
            const uint32_t soff0 = s_lane_off(s_off(rb_req, kb), lane8, kb);
#pragma unroll
            for (int j = 0; j < NJ; ++j) sr[j / 4][j % 4] = ld_s(sign_ptr(0, j), soff0);
        }
    }

    // this lane's column: owning job, tenant (for the scale)
    int myjob[NCT];
    float alpha_m[NCT][kTiledMaxMats];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
        int tenant = 0;
        myjob[ct] = -1;
#pragma unroll
        for (int i = 0; i < kTiledMaxTokens; ++i) {
            myjob[ct] = (c == i && i < a.T[ct]) ? a.col_job[ct][i] : myjob[ct];
            tenant = (c == i && i < a.T[ct]) ? a.col_tenant[ct][i] : tenant;
        }
#pragma unroll
        for (int m = 0; m < kTiledMaxMats; ++m) alpha_m[ct][m] = m < a.n_mats ? a.alpha[m][tenant] : 0.f;
    }

    if (!have_work) return;   // uniform per workgroup (n_rb) / never true for steps (host: waves <= k tiles)
    if constexpr (XSTEPS == 0) {
        // Everything requested so far (the first task's tiles, the scales) has to be there before the first delta job
        // anyway.  Waiting for it here, once, keeps the compiler from putting a wait for a register of the prologue at
        // the top of the task loop, where it would drain the loads in flight at every task.
        __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    }
#pragma unroll
    for (int i = 0; i < (XSTEPS > 0 && !ROOM ? XR : 0); ++i) x_to_operands(xraw[i], xs[i]);
    if constexpr (ROOM) w_turn();
    const uint32_t lanebits = (uint32_t)c << 4;

    // sums of the row blocks in work; accs (8-bit base only): sum_k x of the column, in every row
    float4v accb[RG][NCT], dsel[RG][NCT], accs[NCT];
#pragma unroll
    for (int ct = 0; ct < NCT; ++ct) {
        accs[ct] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int r = 0; r < RG; ++r) accb[r][ct] = dsel[r][ct] = float4v{0.f, 0.f, 0.f, 0.f};
    }
    const half8 ones = __builtin_bit_cast(half8, u32x4{0x3C003C00u, 0x3C003C00u, 0x3C003C00u, 0x3C003C00u});
    // 8 bytes u -> 8 fp16 (1024 + u): byte next to 0x64
    auto q8_operand = [](const u32x4 w2, const int h) {
        const uint32_t lo = w2[2 * h], hi = w2[2 * h + 1];
        return __builtin_bit_cast(half8, u32x4{__builtin_amdgcn_perm(0x64646464u, lo, 0x04010400u),
                                               __builtin_amdgcn_perm(0x64646464u, lo, 0x04030402u),
                                               __builtin_amdgcn_perm(0x64646464u, hi, 0x04010400u),
                                               __builtin_amdgcn_perm(0x64646464u, hi, 0x04030402u)});
    };

    // One task = (row block, k tile, column tile CT).  Its sums are accb[0], dsel[0].  MORE: there is a next task; its tile index is
    // tile_next and its pointers are current (wt, sp).  The base registers are re-requested by the
    // last column tile of a (row block, k tile) only.  xr: this task's x in operand order.  Streamed x, last column tile, new_x (no other
    // row block needs x of this k tile): x of k tile kt_next is fetched, the first column tile's into xnext while this task is
    // multiplied (one column tile: it replaces xr at the end; two: xnext is that tile's own set), the second one's into xr when it is spent.
    // first_rb: the first row block that meets this x (8-bit base: it adds up sum_k x for both).
    // (always_inline on the lambdas: left to its own judgement the compiler may keep one a function, and everything it
    // captures by reference -- every register array of the kernel -- then lives in scratch)
    auto task = [&](auto more_tag, auto ct_tag, u32x4 (&xr)[8], const int kt_cur, const int rb_next, const int kt_next,
                    const bool first_rb, const bool new_x, u32x4 (&xnext)[8]) __attribute__((always_inline)) {
        constexpr bool MORE = decltype(more_tag)::value;
        constexpr int CT = decltype(ct_tag)::value;
        constexpr int CT_NEXT = (CT + 1) % NCT;
        constexpr bool NEW_X = MORE && XSTEPS == 0 && CT == NCT - 1;   // streamed x: if new_x, this task is the last one that needs x of this k tile
        constexpr bool NEW_BASE = CT == NCT - 1;   // the next task is on another tile of W
        // The lane offsets pass through an empty asm in every task: otherwise the compiler hoists
        // "uniform base + lane offset" of every load out of the loop as a 64-bit register pair per load.
        uint32_t l16 = lane16, l8 = lane8;
        asm volatile("" : "+v"(l16), "+v"(l8));
        const uint32_t woff = w_off(rb_next, kt_next) + (ROOM ? 0u : l16), soff = s_lane_off(s_off(rb_next, kt_next), l8, kt_next);
        const unsigned char* const wt_hi = w_base_hi(kt_next);
        const bool short_cur = RM && kt_cur == kt_short;
        // ---- base product; W[v] of the next task goes into the register group just read.  The wavefront runs at a higher
        // priority while it sends these requests (and x's): the other wavefront of the SIMD is in its delta jobs, and a
        // request that waits for an issue slot behind them is a request the memory system gets later (0.3 to 0.7 %).
        __builtin_amdgcn_s_setprio(2);
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            if constexpr (Q8) {
                if constexpr (RM && CT == 0) {   // the first column tile finds the registers as loaded; the second, gathered
                    if ((v & 1) == 0) wr[v >> 1] = rm_gather_q8(wr[v >> 1]);
                }
                accb[0][CT] = __builtin_amdgcn_mfma_f32_16x16x32_f16(q8_operand(wr[v >> 1], v & 1),
                                                                  __builtin_bit_cast(half8, xr[v]), accb[0][CT], 0, 0, 0);
                if constexpr (RG == 1) accs[CT] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, __builtin_bit_cast(half8, xr[v]), accs[CT], 0, 0, 0);
                if constexpr (MORE && NEW_BASE) {
                    if (v & 1) wr[v >> 1] = ld_base(wt_hi, woff, v >> 1);
                }
            } else {
                u32x4 wv = wr[v];
                if (RM && v >= 4) wv = short_cur ? u32x4{0u, 0u, 0u, 0u} : wv;
                accb[0][CT] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, wv),
                                                                  __builtin_bit_cast(half8, xr[v]), accb[0][CT], 0, 0, 0);
                if constexpr (MORE && NEW_BASE) wr[v] = ld_base(wt_hi, woff, v);
            }
            __builtin_amdgcn_sched_barrier(0);   // keep each request behind the MFMA that frees its registers
        }
        if constexpr (Q8 && RG > 1) {
            if (first_rb) {
#pragma unroll
                for (int v = 0; v < 8; ++v) accs[CT] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, __builtin_bit_cast(half8, xr[v]), accs[CT], 0, 0, 0);
            }
        }
        if constexpr (NEW_X) {
            if (RG == 1 || new_x) x_fetch_operands(xnext, kt_next, 0);
        }
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
        // ---- delta jobs.  The 8 NJ (job, slice) pairs of the task form one sequence; the table
        // look-up of pair i + kLookAhead is issued before the MFMA of pair i, through a ring of
        // operand registers, and a job's sign words are re-requested as soon as its last address exists.
        // (row-major with many jobs and resident x: a shorter ring, so that nothing ends up in scratch.  Measured with rings of 4 to 14 look-ups ahead: the depth does not change the time of a task.)
        constexpr int kLookAhead = RM && XSTEPS > 0 && (ROOM ? NJ >= 10 && XSTEPS == 2 : NJ == 16) ? 4 : 6, kRing = kLookAhead + 2, kPairs = 8 * NJ;
        u32x4 ring[kRing];
        float4v sel = {0.f, 0.f, 0.f, 0.f};   // the job owning this lane's column, this tile
        auto look_up = [&](const int i) __attribute__((always_inline)) {      // i = 8 * job + slice
            const int j = i >> 3, v = i & 7;
            if constexpr (S4) {
                if (v == 0 && j % 4 == 0) turn_s4(sr[j / 4]);
            } else if constexpr (RM) {
                if (v == 0) sr[j / 4][j % 4] = rm_gather_sign_bytes(sr[j / 4][j % 4]);
            }
            ring[i % kRing] = RM && !S4 ? lut_read_rm(sr[j / 4][j % 4], v, lanebits) : lut_read(sr[j / 4][j % 4], v, lanebits);
            if constexpr (MORE && S4) {
                if (v == 7 && (j % 4 == 3 || j == NJ - 1)) ld_s4(sr[j / 4], CT_NEXT, j / 4, kt_next);
            } else if constexpr (MORE) {
                if (v == 7) sr[j / 4][j % 4] = ld_s(sign_ptr(CT_NEXT, j), soff);
            }
        };
#pragma unroll
        for (int i = 0; i < kLookAhead; ++i) look_up(i);
        float4v acc = {0.f, 0.f, 0.f, 0.f};
        auto finish_job = [&](const int j) __attribute__((always_inline)) {
            const bool mine = (myjob[CT] == j);
#pragma unroll
            for (int q = 0; q < 4; ++q) sel[q] = mine ? acc[q] : sel[q];
            // pin the selection here: left alone, the compiler sinks all of them below the last job
            // and keeps one live accumulator per job
            asm volatile("" : "+v"(sel[0]), "+v"(sel[1]), "+v"(sel[2]), "+v"(sel[3]));
            acc = float4v{0.f, 0.f, 0.f, 0.f};
            __builtin_amdgcn_sched_barrier(0);
        };
        auto pair = [&](const int i) __attribute__((always_inline)) {
            if (i + kLookAhead < kPairs) look_up(i + kLookAhead);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, ring[i % kRing]),
                                                         __builtin_bit_cast(half8, xr[i & 7]), acc, 0, 0, 0);
        };
        if constexpr (S4 || ROOM) {
            // Two loops, unrolled from the inside: as one of 128 iterations it is too large for the compiler to unroll once the
            // row-major exchanges are in it, and the operands then live in scratch.
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                if constexpr (MORE && NEW_BASE && ROOM) {   // the next base tile has arrived: the last job hides its trip through LDS
                    if (j == NJ - 1) w_turn();
                }
#pragma unroll
                for (int v = 0; v < 8; ++v) pair(8 * j + v);
                finish_job(j);
            }
        } else {
#pragma unroll
            for (int i = 0; i < kPairs; ++i) {
                pair(i);
                if ((i & 7) == 7) finish_job(i >> 3);
            }
        }
        dsel[0][CT] += sel;
        if constexpr (NEW_X) {
            if (RG == 1 || new_x) {
                if constexpr (NCT == 1) {   // this task's x is spent: move the next one in
#pragma unroll
                    for (int v = 0; v < 8; ++v) {
                        // (moves that stay here: as plain copies they sink behind the join with the path on which a row block ends, where the
                        // compiler waits for every load in flight.  Identity permutations are not moved across control flow.)
                        u32x4 t;
#pragma unroll
                        for (int i = 0; i < 4; ++i) t[i] = (uint32_t)__builtin_amdgcn_mov_dpp((int)xnext[v][i], 0xE4, 0xF, 0xF, true);
                        xr[v] = t;
                    }
                } else {
                    x_fetch_operands(xr, kt_next, 1);
                }
            }
        }
    };

    // The partial tiles of `n` finished row blocks, first one rbg0: add the wavefronts in a fixed order, write y.
    auto flush = [&](const int rbg0, const int n, const bool more_follow) __attribute__((always_inline)) {
        __syncthreads();
        for (int idx = threadIdx.x; idx < n * 256; idx += blockDim.x) {   // n slots = n / NCT row blocks
            const int slot = idx >> 8, e = idx & 255, col = e >> 4, row = e & 15;
            const int ct = slot % NCT;
            int m, rb;
            mat_of(rbg0 + slot / NCT, m, rb);
            const int out = a.out[m], n_row = rb * kTileRows + row;
            const u32x2 meta = *(const u32x2*)(smem + Plan::kMeta + (ct * kTiledMaxTokens + col) * 8);
            const int span = (int)meta[0];   // columns of this token (its planes); 0: not a token's first column
            if (col < a.T[ct] && n_row < out && span > 0) {
                float s = 0.f;
                for (int p = 0; p < span; ++p)
                    for (int wv = 0; wv < nw; ++wv)
                        s += *(const float*)(smem + kLutBytes + wv * Plan::kRegion + (slot * 256 + e + p * 16) * 4);
                a.y[m][(int64_t)(int)meta[1] * out + n_row] = f2h_rne(s);
            }
        }
        if (more_follow) {
            // The stores of y must not be outstanding when the task loop goes on: loads and stores share one counter,
            // and with both kinds in flight the compiler can only wait for all of them -- it would put that wait at
            // the top of the task loop, where it drains the requested tiles at every task.
            if constexpr (XSTEPS == 0) __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
            __syncthreads();
        }
    };

    int slot = 0, flush_base = r0;
    int m_cur = m_req;
    int rbi = 0;            // the first row block being multiplied: r0 + rbi
    int pair = 0;           // 1: the one after it as well
    bool last_rb = false;   // they are the last ones
    float4v sc[RG];         // 8-bit base: the scales of this lane's 4 output rows, asked for long before their use
    int m_nx = m_req, rb_nx = 0;         // where the requests go after the last task of these row blocks
    auto begin_rb = [&]() __attribute__((always_inline)) {
        if constexpr (RG == 2) pair = r0 + rbi + 1 < min(r1, a.rb_end[m_cur]) ? 1 : 0;
        last_rb = rbi + pair + 1 == n_rb;
        if constexpr (Q8) {
            const float* ws = m_cur == 0 ? a.wscale[0] : (m_cur == 1 ? a.wscale[1] : a.wscale[2]);
#pragma unroll
            for (int r = 0; r < RG; ++r) {
                const int rb = rb_req + (r ? pair : 0);
                if constexpr (RM) {   // the caller's array of `out` scales: rows beyond `out` read the last one (never stored)
#pragma unroll
                    for (int i = 0; i < 4; ++i) sc[r][i] = ws[min(rb * kTileRows + 4 * g + i, a.out[0] - 1)];
                } else {
                    sc[r] = *(const float4v*)(ws + rb * kTileRows + 4 * g);   // the scale array is padded to whole row blocks
                }
            }
        }
        m_nx = m_req;
        rb_nx = 0;
        if (!last_rb) mat_of(r0 + rbi + pair + 1, m_nx, rb_nx);
    };
    auto cross = [&]() __attribute__((always_inline)) {   // requests move on to the next row block: switch the pointers if it is in another matrix
        if constexpr (RM) rm_lane_offsets(rb_nx);
        if (m_nx != m_req) {
            wt = (const unsigned char*)a.wt[m_nx];
#pragma unroll
            for (int ct = 0; ct < NCT; ++ct)
#pragma unroll
                for (int j = 0; j < NJ; ++j) sp[ct][j] = (const unsigned char*)a.signs[ct][m_nx][j];
        }
    };
    // a row block is done: this wavefront's partial tiles -> slots; the slots are added up and written when they are full
    // more_tag: std::true_type / std::false_type where the caller knows whether another one follows these, RbDynamic where last_rb tells
    struct RbDynamic {};
    auto end_rb = [&](auto r_tag, auto more_tag) __attribute__((always_inline)) {
        constexpr int r = decltype(r_tag)::value;
        bool last;
        if constexpr (std::is_same<decltype(more_tag), RbDynamic>::value) last = last_rb;
        else last = !decltype(more_tag)::value && (RG == 1 || r == pair);
#pragma unroll
        for (int ct = 0; ct < NCT; ++ct) {
            const float al = m_cur == 0 ? alpha_m[ct][0] : (m_cur == 1 ? alpha_m[ct][1] : alpha_m[ct][2]);
            float4v p = accb[r][ct];
            if constexpr (Q8) {
#pragma unroll
                for (int i = 0; i < 4; ++i) p[i] = sc[r][i] * (accb[r][ct][i] - 1152.f * accs[ct][i]);
            }
            if (a.planes > 1) {   // several planes per token: only a token's first column carries the base product
                const int span = *(const int*)(smem + Plan::kMeta + (ct * kTiledMaxTokens + c) * 8);
                if (span == 0) p = float4v{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) p[i] += al * dsel[r][ct][i];
            *(float4v*)(region + ((slot + ct) * 256 + c * 16 + 4 * g) * 4) = p;   // [column][row]
            accb[r][ct] = dsel[r][ct] = float4v{0.f, 0.f, 0.f, 0.f};
            if (XSTEPS > 0) accs[ct] = float4v{0.f, 0.f, 0.f, 0.f};
        }
        slot += NCT;
        if (slot == Plan::kRedSlots || last) {
            flush(flush_base, slot, !last);
            flush_base += slot / NCT;
            slot = 0;
        }
    };
    auto next_rb = [&]() __attribute__((always_inline)) {
        m_cur = m_nx;
        m_req = m_nx;
        rb_req = rb_nx;
        rbi += 1 + pair;
    };
    using I0 = std::integral_constant<int, 0>;
    using CtL = std::integral_constant<int, NCT - 1>;
    if constexpr (XSTEPS > 0) {
        while (rbi < n_rb) {
            begin_rb();
#pragma unroll
            for (int ki = 0; ki < XSTEPS; ++ki) {
                if (ki + 1 < XSTEPS) {
                    task(std::true_type{}, I0{}, xs[ki], kb + ki * kstride, rb_req, kb + (ki + 1) * kstride, true, false, xraw[0]);
                } else if (!last_rb) {
                    cross();
                    task(std::true_type{}, I0{}, xs[ki], kb + ki * kstride, rb_nx, kb, true, false, xraw[0]);
                } else {
                    task(std::false_type{}, I0{}, xs[ki], kb + ki * kstride, 0, 0, true, false, xraw[0]);
                }
            }
            end_rb(I0{}, RbDynamic{});
            next_rb();
        }
    } else {
        // Streamed x: ONE loop over all (k tile, row block) pairs but the last, with a single copy of the task that requests its
        // successor, and the last one after the loop.  (As a loop nest with the last task inside it, the compiler
        // kept two sets of registers for the requested tiles, copied one into the other at the end of every task and
        // waited there for every outstanding load: nothing was in flight across a task boundary.)
        begin_rb();
        int ki = 0, r = 0;
        auto first_column_tile = [&]() __attribute__((always_inline)) {   // all but the last column tile: the next task stays on this tile
            if constexpr (NCT == 2) task(std::true_type{}, I0{}, xs[0], kb + ki * kstride, rb_req + r, kb + ki * kstride, r == 0, false, xraw[0]);
        };
        auto other_row_block = [&]() __attribute__((always_inline)) {     // accb[0], dsel[0] are the sums of row block r
            if constexpr (RG == 2) {
                if (pair) {
#pragma unroll
                    for (int ct = 0; ct < NCT; ++ct) {
                        const float4v b0 = accb[0][ct], d0 = dsel[0][ct];
                        accb[0][ct] = accb[RG - 1][ct];
                        dsel[0][ct] = dsel[RG - 1][ct];
                        accb[RG - 1][ct] = b0;
                        dsel[RG - 1][ct] = d0;
                    }
                    r ^= 1;
                }
            }
        };
        auto end_all = [&](auto more_tag) __attribute__((always_inline)) {
            end_rb(I0{}, more_tag);
            if constexpr (RG == 2) {
                if (pair) end_rb(std::integral_constant<int, 1>{}, more_tag);
            }
        };
        for (int t = n_rb * steps; t > 1; --t) {
            const int kt = kb + ki * kstride;
            const bool last_r = RG == 1 || r == pair, done = last_r && ki + 1 == steps;
            first_column_tile();
            if (done) cross();
            else if constexpr (RM && RG == 2) rm_lane_offsets(rb_req + (last_r ? 0 : 1));
            task(std::true_type{}, CtL{}, xs[NCT - 1], kt, done ? rb_nx : rb_req + (last_r ? 0 : 1), !last_r ? kt : done ? kb : kt + kstride,
                 r == 0, last_r, NCT == 2 ? xs[0] : xraw[0]);
            other_row_block();
            ki += last_r ? 1 : 0;
            if (done) {
                end_all(std::true_type{});
#pragma unroll
                for (int ct = 0; ct < NCT; ++ct) accs[ct] = float4v{0.f, 0.f, 0.f, 0.f};
                next_rb();
                begin_rb();
                ki = 0;
            }
        }
        first_column_tile();
        task(std::false_type{}, CtL{}, xs[NCT - 1], kb + ki * kstride, 0, 0, r == 0, false, xraw[0]);
        other_row_block();
        end_all(std::false_type{});
    }
}

template <bool Q8, bool RM, int NJ, int XSTEPS, int NCT = 1, bool S4 = RM, int RG = 1>
static hipError_t launch_inst(const TiledArgs& args, int n_waves, unsigned grid, hipStream_t st) {
    auto kernel = linear_decode_tiled_kernel<NJ, XSTEPS, NCT, Q8, RM, S4, RG>;
    const size_t lds = (size_t)LdsPlan<XSTEPS, rm_base_through_lds(NJ, XSTEPS, Q8, RM)>::kTotal;
    static PerDeviceOnce lds_limit;   // one per instantiation
    const hipError_t ea = lds_limit.run([&] {
        hipFuncAttributes fa;
        const hipError_t e = hipFuncGetAttributes(&fa, (const void*)kernel);
        if (e != hipSuccess) return e;
        if (fa.sharedSizeBytes != 0) return hipErrorInvalidValue;   // the table must start at LDS address 0
        return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    });
    if (ea != hipSuccess) return ea;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(n_waves * kWave), lds, st, args);
    return hipGetLastError();
}

template <bool Q8, bool RM, int NJ>
static hipError_t launch_nj(const TiledArgs& args, int n_waves, int xsteps, unsigned grid, int rounds, int cus, hipStream_t st) {
    // Row-major: the signs slot by slot (see S4) where that is the better one, both measured with the tensors coming from HBM (180
    // + 260 + 290 launches of 2 to 32 tenants).  Four slots at a time issue half the loads, but ask L2 twice for a row's 32 bytes, and the second
    // time the line may be gone: with long rows, with several row blocks per workgroup, and where rows of signs do not start on 128-byte
    // lines (in % 1024 != 0), so that neighbouring k tiles share lines.  4 at a time / slot by slot, us:
    //   one column tile, 11008 x 11008, 8 slots 109 / 93; 11008 x 5120, 16 slots 84 / 73; 4096 x 5760, 8 slots 24.2 / 23.0; 2500 x 5120,
    //     12 slots 22.0 / 22.7; 8192 x 2304, 12 slots 24.0 / 25.2; 8-bit base, 11008 x 11520, 4 slots 69 / 64
    //   two, 32 tenants: 11008 x 3328 94 / 85; 8192 x 2048 40 / 44; 4096 x 4096 40 / 42; 6000 x 5120 88 / 84; 2500 x 5760 (8-bit base) 52 / 47
    const bool several = args.rb_end[args.n_mats - 1] > (int)grid;
    const int KT = args.KT;
    // Streamed x: two row blocks at a time (RG) where workgroups have several, rows are long and x is a large part of what a task asks for.  One
    // at a time / two, us, weights from HBM:
    //   one column tile, 12 and 16 slots, a 70B layer's 28672 x 8192: 141 / 135 and 171 / 160, 8-bit base 123 / 115 and 155 / 145, row-major 189 / 178 and
    //     229 / 218; 8 slots, 5120 x 5120 21.2 / 20.0, 8-bit base 8192 x 3328 1.06 x, 12288 x 3328 0.98 to 0.99 x; 12000 rows of 2496 and fewer 0.97 to 1.00 x
    //   4 and 6 slots, 28672 x 8192: 8-bit base 65.3 / 63.5 and 80.0 / 76.0, row-major 120.8 / 117.5 and 136 / 131, row-major over the 8-bit base 95.9 / 88.7 and
    //     115 / 107; 12000 rows of 704 to 7104 0.97 to 0.99 x
    //   two: 5 tenants, 20 tokens: 28672 x 8192 147 / 128, 8192 x 3584 25.1 / 23.4, 12000 x 2496 29.4 / 29.7, 12000 x 1216 21.6 / 22.8; 24 and 32 tenants:
    //     28672 x 8192 239 / 224, 12000 x 1280 34.9 / 33.6 and 41.1 / 40.4, row-major 5120 x 2304 43.4 / 41.3, but 12000 x 640 42.8 / 43.8
    // Few slots over the fp16 base ask for little but weights, and where nearly all units have a workgroup the memory sets the time: 8192 x 8192
    // and 28672 x 8192 with 4 slots 31.9 / 32.8 and 96.0 / 97.8, row-major 8192 x 8192 43.8 / 44.8; with 8 slots 12288 x 4608 (a row block is left over) 0.98 x.
    // Where a fifth of the units is idle the others' requests are the limit: 5120 x 8192 4, 6 and 8 slots 1.06, 1.08 and 1.10 x.
    const bool full = 5 * (int)grid > 4 * cus;
    const bool pays = Q8 || !full || (RM ? NJ > 4 || rounds > 2 : NJ > 8 || (NJ == 8 && rounds != 3));
    const bool two = several && (args.n_ct == 2 ? KT >= (NJ >= 12 ? 5 : 12) : pays && KT >= (NJ >= 8 ? 12 : 30));
    auto streamed = [&](auto nct_tag, auto s4_tag) {
        constexpr int NCT = decltype(nct_tag)::value;
        constexpr bool S4 = decltype(s4_tag)::value;
        if constexpr (NJ > 2 || NCT == 2) {
            if (two) return launch_inst<Q8, RM, NJ, 0, NCT, S4, 2>(args, n_waves, grid, st);
        }
        return launch_inst<Q8, RM, NJ, 0, NCT, S4>(args, n_waves, grid, st);
    };
    using One = std::integral_constant<int, 1>;
    using Two = std::integral_constant<int, 2>;
    if constexpr (RM && (NJ > 4 || (Q8 && NJ == 4))) {
        const bool split_lines = args.in % 1024 != 0;
        if (xsteps == 0 && args.n_ct == 1 &&
            (NJ > 4 ? KT > 24 || (KT > 16 && split_lines) || (KT > 12 && several) : (KT > 16 && split_lines) || (KT > 32 && several)))
            return streamed(One{}, std::false_type{});
        if constexpr (NJ > 4) {
            if (args.n_ct == 2 && (KT > 24 || (KT > 16 && (split_lines || (several && NJ > 6))) || (KT > 12 && split_lines && NJ > (several ? 6 : 8))))
                return streamed(Two{}, std::false_type{});
        }
    }
    if (args.n_ct == 2) return streamed(Two{}, std::bool_constant<RM>{});   // 17..32 tokens: two column tiles, streamed x
    if (xsteps == 1) return launch_inst<Q8, RM, NJ, 1>(args, n_waves, grid, st);
    if (xsteps == 2) return launch_inst<Q8, RM, NJ, 2, 1, RM && (Q8 || NJ <= 12)>(args, n_waves, grid, st);
    return streamed(One{}, std::bool_constant<RM>{});
}

template <bool Q8, bool RM = false>
static hipError_t launch_tiled_t(const TiledArgs& args, int n_jobs, hipStream_t st) {
    if (RM && (args.n_mats != 1 || args.in % 128 != 0 || args.in < 128 || !args.packed_by_tenant)) return hipErrorInvalidValue;
    if (n_jobs < 1 || n_jobs > kTiledMaxJobs || args.n_mats < 1 || args.n_mats > kTiledMaxMats || args.n_ct < 1 ||
        args.n_ct > kTiledMaxCt)
        return hipErrorInvalidValue;
    const int rb_total = args.rb_end[args.n_mats - 1];
    if (rb_total < 1 || args.KT < 1) return hipErrorInvalidValue;
    // compute units of the current device, asked once per device (0 = not asked yet; 64 devices at most are remembered)
    static std::atomic<int> cus_of[64];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return hipErrorInvalidDevice;
    int cus = cus_of[dev & 63].load(std::memory_order_relaxed);
    if (cus == 0) {
        int v = 0;
        cus = (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) ? v : 256;
        cus_of[dev & 63].store(cus, std::memory_order_relaxed);
    }
    // Persistent grid: at most one workgroup per compute unit, never more workgroups than row blocks -- and of the
    // grids that need the same number of rounds (row blocks per workgroup, rounded up) the SMALLEST: 1376 row blocks
    // (gate,up of Llama-2-7B) on 256 units are 6 rounds either way, but 256 workgroups leave 160 units idle during the
    // sixth while 230 workgroups of 6 (four of them 5) keep all of theirs streaming to the end.  The launch is bound by
    // HBM, not by the number of units, so it then takes the time of 5.4 rounds instead of 6.
    // 8 wavefronts, never more than k tiles (an empty reduction, KT == 0, never gets here: the host writes y = 0)
    const int rounds = (rb_total + cus - 1) / cus;
    const unsigned grid = (unsigned)((rb_total + rounds - 1) / rounds);
    int n_waves = kMaxWavesTiled;
    while (n_waves > 1 && n_waves > args.KT) n_waves >>= 1;
    int xsteps = 0;
    if (args.KT > 0 && args.KT % n_waves == 0 && args.KT / n_waves <= 2) xsteps = args.KT / n_waves;
    auto go = [&](auto nj) {
        return launch_nj<Q8, RM, decltype(nj)::value>(args, n_waves, args.n_ct == 2 ? 0 : xsteps, grid, rounds, cus, st);
    };
    // A slot without a job costs as much as one with: its signs are requested (slot 0's again) and looked up.  With slots for 4, 8
    // or 16 only, a 7B layer took 142 us with 9 tenants and 149 with 12 (134 and 139 over the 8-bit base); in steps of two it
    // takes 125 and 137 (103 and 117).
    if (n_jobs <= 2) return go(std::integral_constant<int, 2>{});
    if (n_jobs <= 4) return go(std::integral_constant<int, 4>{});
    if (n_jobs <= 6) return go(std::integral_constant<int, 6>{});
    if (n_jobs <= 8) return go(std::integral_constant<int, 8>{});
    if (n_jobs <= 10) return go(std::integral_constant<int, 10>{});
    if (n_jobs <= 12) return go(std::integral_constant<int, 12>{});
    if (n_jobs <= 14) return go(std::integral_constant<int, 14>{});
    return go(std::integral_constant<int, 16>{});
}

}  // namespace bd

// kernels.hpp -- gfx950 kernels of one Swendsen-Wang sweep and of connected-
// component labeling on a 2D square lattice.
//
// A sweep is three launches (Sec. II: T_SW = T_activate + T_identify + T_flip,
// with T_identify = T_local + T_global):
//
//   k_tile    one workgroup per 128x64 tile.  Bond activation (Sec. II.A) fused
//             with tile labeling (Sec. II.B): each lane of a 64-lane wave owns
//             two sites of a tile row; the row's bonds become 128-bit masks by
//             wave ballots, right bonds turn into row runs (each site's run
//             start from a DPP max-scan over the lanes), each run takes the
//             label of one run above it as its wave goes down its rows, and the
//             down bonds left over (a run touching several labels, or another
//             wave's rows) join labels by a lock-free union-find in LDS, fed
//             from compacted per-wave lists.
//             Clusters that touch the tile border are claimed by their border
//             sites and get a compact boundary id; every site's result is a
//             16-bit code (the slot of its interior root, or TSITES + boundary id).
//   k_merge   tile consolidation (Sec. II.C) in one pass: every active bond
//             that crosses a tile edge, the periodic wrap included, unites two
//             boundary ids in a global union-find over the compact id space
//             (CAS linking of the larger-key root under the smaller one).  Only
//             ~2(TW+TH) ids per tile exist, so this structure stays small and
//             cache resident.
//   k_flatten resolves every boundary id to its root, whose key is the
//             cluster's minimum site index (the canonical label), draws one new
//             state per cluster from that root (Sec. II.D) and writes spins
//             and, optionally, labels.
//
// Labeling-only inputs (packed bond bytes or binary images) reuse the same
// three kernels with a different bond source.  The few-cluster update
// (Sec. III) labels with the same tile and merge launches, marks the clusters
// that hold a seed in k_seed and flips only those in k_flatten<M_FEW>.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "philox.hpp"
#include "uf.hpp"

namespace swccl {

constexpr int TW = 128;               // tile width: a wave covers a tile row, 2 sites per lane
constexpr int RPW = 8;                // tile rows per wave
constexpr int TLIST = 3 * TW;         // k_tile's per-wave lists: a row adds at most TW entries, a
                                      // fuller list is worked off first (keeps the LDS per wave small)
constexpr uint16_t ID_NONE = 0xFFFF;
constexpr uint16_t CODE_BG = 0xFFFF;

// Tile shapes: TW x TH sites, one wave per RPW rows, so a tile is worked by
// TH / RPW waves.  Per tile there are CAP boundary ids (at least the border
// sites), EDGE edge entries (top row, bottom row, left column, right column)
// and XW words of crossing bits (the right edge's rows, XR words of 64, then
// the bottom edge's even and odd columns).
template <int TH_>
struct Tile {
    static constexpr int TH = TH_;
    static constexpr int TSITES = TW * TH;
    static constexpr int CAP = 2 * (TW + TH);
    static constexpr int EDGE = 2 * TW + 2 * TH;
    static constexpr int XR = (TH + 63) / 64;
    static constexpr int XW = XR + 2;
    static constexpr int NWAVE = TH / RPW;
    static constexpr int NT = 64 * NWAVE;
    static_assert(TH % RPW == 0 && TH >= 2 * RPW && TH <= 128, "tile heights 16, 32, 64, 128");
    static_assert(CAP + TSITES < 0xFFFE, "codes are 16-bit");
};
constexpr int TH_DEFAULT = 64;        // the shape the library uses unless told otherwise

// Kernels that do not depend on the tile shape run 512-thread workgroups.
constexpr int NT = 512;
constexpr int NWAVE = NT / 64;

// The one-tile lattices that k_small sweeps whole in LDS: W <= 128, H <= 64.
constexpr int SMALL_W = 128, SMALL_H = 64, SMALL_SITES = SMALL_W * SMALL_H;

enum : uint32_t { TAG_INIT = 0, TAG_BOND = 1, TAG_FLIP = 2, TAG_SEED = 3, TAG_FEW = 4 };
// M_FEW is a flatten mode only: the few-cluster update labels with M_SW's
// tile and merge kernels and flips in k_flatten<M_FEW>.
enum Mode : int { M_SW = 0, M_BONDS_PERIODIC = 1, M_BONDS_OPEN = 2, M_SITES = 3, M_FEW = 4 };

// Observable counters (unsigned 64-bit, two's complement for signed values),
// and the observables' workgroup ticket.
enum { ST_ACTIVE = 0, ST_NCLUST = 1, ST_NSAT = 2, ST_MAGNET = 3, ST_COUNTS = 4, ST_DIGEST = 12, ST_TICKET = 15,
       ST_LEN = 16 };

struct Grid {
    int W, H, ntx, nty, ntiles;
    int rev;  // visit the tiles in reverse order (single lattices only; a schedule check)
};

// One lattice of a batched launch (many independent lattices swept by one
// launch per phase): its shape, buffers and random-number parameters, and the
// first of its tiles in the batch's tile arrays.
struct LatticeDesc {
    Grid g;
    int32_t tile0;
    uint8_t *spins;
    uint8_t *bonds;    // packed bonds of the sweep, or nullptr
    int32_t *labels;   // canonical labels, or nullptr
    uint32_t tm1, tany, k0, k1, sid, q;
    int32_t ising;
    int32_t nmerge;    // fused sweeps: merge groups of the lattice (0 if swept whole in LDS)
};

// How a batched launch finds the lattice of a tile.  Tile-indexed arrays
// (codes, ids, edges, ...) are concatenated over the batch and indexed by the
// batch tile; geometry uses the tile's index inside its lattice.
struct Batch {
    const LatticeDesc *lat;
    const int32_t *lat_of_tile;  // batch tile -> lattice
    const uint32_t *t;           // the batch's sweep counter, read on the device (graph replays)
    int32_t tile_base, ntiles;   // this launch covers tiles [tile_base, tile_base + ntiles)
};

// Shared device helpers (XCD placement, lane masks, union-find in LDS and
// over global ids, wave reductions) are in uf.hpp.

// ----------------------------------------------------------------- init ----

// Initial states: state_i = (w q) >> 32 with w = Philox(i>>2, 0, INIT, sid)[i&3].
__global__ __launch_bounds__(NT) void k_init(uint8_t *spins, int64_t N, uint32_t q, int ising,
                                             uint32_t k0, uint32_t k1, uint32_t sid)
{
    const int64_t w = static_cast<int64_t>(blockIdx.x) * NT + threadIdx.x;
    const int64_t base = w * 4;
    if (base >= N) return;
    const U4 b = philox4x32_10(static_cast<uint32_t>(w), 0u, TAG_INIT, sid, k0, k1);
    const uint32_t words[4] = {b.v0, b.v1, b.v2, b.v3};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (base + j < N) {
            const uint32_t st = draw_state(words[j], q);
            spins[base + j] = ising ? static_cast<uint8_t>(2 * st - 1) : static_cast<uint8_t>(st);
        }
    }
}

__global__ void k_zero_u64(unsigned long long *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}

__global__ void k_zero_i32(int32_t *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

// Copy n bytes from host memory the device can read (pinned) into device
// memory, in the compute queue: a small request's image and a batch's table
// then never wait behind large copies queued on the copy engines.  16 bytes a
// thread, in one load where both addresses are multiples of 16.
constexpr int PULL = 16;
__global__ __launch_bounds__(NT) void k_pull(uint8_t *dst, const uint8_t *src, int64_t n)
{
    const int64_t i = (static_cast<int64_t>(blockIdx.x) * NT + threadIdx.x) * PULL;
    const bool whole = ((reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src)) & (PULL - 1)) == 0;
    if (whole && i + PULL <= n) {
        *reinterpret_cast<uint4 *>(dst + i) = *reinterpret_cast<const uint4 *>(src + i);
    } else {
#pragma unroll
        for (int j = 0; j < PULL; ++j)
            if (i + j < n) dst[i + j] = src[i + j];
    }
}

__global__ void k_iota_i32(int32_t *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = i;
}

// Advance a device-side sweep counter (the last launch of a batched sweep).
__global__ void k_bump_u32(uint32_t *p)
{
    if (threadIdx.x == 0) p[0] += 1u;
}

// ----------------------------------------------------------------- tile ----

struct TileArgs {
    Grid g;
    const uint8_t *in;        // spins (M_SW), packed bonds or image bytes
    uint8_t *bonds_out;       // M_SW: packed bonds of this sweep, or nullptr
    uint16_t *codes;          // [ntiles][TSITES]
    int32_t *gkey;            // [ntiles][CAP]
    int32_t *gparent;         // [ntiles][CAP]
    int32_t *gsize;           // [ntiles][CAP] or nullptr (zeroed here when given)
    uint16_t *edges;          // [ntiles][EDGE]
    uint64_t *xbits;          // [ntiles][XW]
    int32_t *nb;              // [ntiles]
    int32_t *tile_act;        // [ntiles]: active bonds owned by the tile (M_SW)
    uint32_t tm1;             // M_SW: a bond is active iff its word r <= tm1 ...
    uint32_t tany;            // ... and tany (threshold T > 0); tm1 = T - 1
    uint32_t k0, k1, t, sid;
    Batch b;                  // batched launches only
    uint32_t rk[20];          // single-lattice sweeps: the Philox key schedule of (k0, k1), round r in
                              // rk[2r], rk[2r + 1]
};

// Wave-uniform copy of a mask read from LDS.
__device__ __forceinline__ uint64_t uniform64(uint64_t v)
{
    const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v));
    const uint32_t hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(v >> 32));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}
// A pointer the caller knows to be wave-uniform, as a scalar value.
template <typename T>
__device__ __forceinline__ T *uniform_ptr(T *p)
{
    return reinterpret_cast<T *>(static_cast<uintptr_t>(uniform64(static_cast<uint64_t>(reinterpret_cast<uintptr_t>(p)))));
}

// Border position t of a tile in the layout of the edge arrays: top row,
// bottom row, left column, right column.  Returns the slot, or -1 if the
// position lies outside a ragged tile.
template <int TH>
__device__ __forceinline__ int border_slot(int t, int tw, int th)
{
    if (t < TW) return t < tw ? t : -1;
    if (t < 2 * TW) return (t - TW) < tw ? (th - 1) * TW + (t - TW) : -1;
    if (t < 2 * TW + TH) return (t - 2 * TW) < th ? (t - 2 * TW) * TW : -1;
    return (t - 2 * TW - TH) < th ? (t - 2 * TW - TH) * TW + tw - 1 : -1;
}

// A site's 16-bit code: the slot of its cluster's root inside the tile
// (0 .. TSITES - 1), or TSITES + k for the cluster of boundary id k, or
// CODE_BG.

// Maximum of v over the lanes below the calling one (0 for lane 0), v >= 0:
// an inclusive max-scan by row shifts and row broadcasts, then a shift by one
// lane.  Out-of-row sources read 0, the identity; rows outside a broadcast's
// row mask keep their value.
__device__ __forceinline__ int wave_max_below(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false));  // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false));  // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false));  // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false));  // row_shr:8
    // The row broadcasts write only the rows in their masks (1 and 3, then 2
    // and 3) and leave the others as they are: with the destination as the
    // second source that is one max per step (the compiler emits a copy, a
    // broadcast and a max).  s_nop 1 gives each DPP read of a just-written
    // register its two wait states.
    int out;
    asm("s_nop 1\n\t"
        "v_max_i32_dpp %0, %0, %0 row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_i32_dpp %0, %0, %0 row_bcast:31 row_mask:0xc bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_mov_b32_dpp %1, %0 wave_shr:1 row_mask:0xf bank_mask:0xf bound_ctrl:1"  // lane 0 reads 0
        : "+v"(v), "=v"(out));
    return out;
}

// LDS of the tile phase, a 128 x 64 tile: 39 KB with eight rows a wave (eight
// lists), 45 KB with four (sixteen).  A CU holds 32 waves of these kernels (8 a
// SIMD), which share its 160 KB: LDS_PER_WAVE each.
constexpr size_t LDS_PER_WAVE = 160 * 1024 / 32;
template <int MODE, int TH_, int RPW_ = RPW>
struct TileSmem {
    static constexpr int TH = TH_, TSITES = TW * TH, NWAVE = TH / RPW_;
    alignas(8) int P[TSITES + 4];      // union-find parent per site slot, as 4 x slot; P[TSITES]: background
    uint16_t wl[NWAVE][TLIST];         // per-wave work list (contacts, then linked labels)
    uint32_t xr_w[NWAVE];              // right crossing bonds of each wave's rows (bit r: its row r)
    EO xd_s;                           // bottom crossing bonds
    int nb_s;
    int act_w[NWAVE];
};
template <int MODE, int TH_, int RPW_>
constexpr bool tile_fits = sizeof(TileSmem<MODE, TH_, RPW_>) <= LDS_PER_WAVE * (TH_ / RPW_);

// A batched launch's tile: take the lattice's shape, buffers and keys from
// its descriptor; lt is the tile's index inside its lattice.
__device__ __forceinline__ void load_batch_tile(TileArgs &a, int tile, int &lt)
{
    const LatticeDesc &L = a.b.lat[a.b.lat_of_tile[tile]];
    a.g = L.g;
    a.in = L.spins;
    a.bonds_out = L.bonds;
    a.tm1 = L.tm1;
    a.tany = L.tany;
    a.k0 = L.k0;
    a.k1 = L.k1;
    a.sid = L.sid;
    a.t = *a.b.t;
    lt = tile - L.tile0;
}

// The kernel's own TileArgs in the kernel-argument segment, behind an opaque
// copy of the segment pointer: a field read through it is a scalar load at
// that point, so output pointers used only at the end of the tile phase are
// not held in scalar registers across it (which would spill some).
typedef const __attribute__((address_space(4))) TileArgs KernTileArgs;
__device__ __forceinline__ KernTileArgs *kernel_tile_args()
{
    KernTileArgs *k = (KernTileArgs *)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(k));
    return k;
}

// The tile phase of one tile: `tile` indexes the tile arrays, `lt` is the
// tile inside its lattice (they differ in batches).  Uses every thread of a
// Tile<TH>::NT-thread workgroup; ends with the workgroup's writes issued.
// With KARG the launch's only argument is the TileArgs `a` came from, and the
// output pointers are re-read from it where they are used; with RKEYS (a
// single-lattice sweep) so is the bond generator's key schedule, row by row
// (scalar loads in place of 18 scalar adds per row).
template <int MODE, bool EVENW, int TH_, bool KARG = false, bool RKEYS = false, int RPW_ = RPW>
__device__ __forceinline__ void tile_body(TileArgs a, const int tile, const int lt, TileSmem<MODE, TH_, RPW_> &sm)
{
    using S = Tile<TH_>;
    constexpr int TH = S::TH, TSITES = S::TSITES, CAP = S::CAP, EDGE = S::EDGE, XR = S::XR, XW = S::XW;
    constexpr int RPW = RPW_, NWAVE = TH / RPW, NT = 64 * NWAVE;  // rows per wave
    constexpr bool NEED_DOWN = MODE == M_SW || MODE == M_SITES;  // bonds from two rows
    constexpr bool NEED_HALO = MODE == M_SW || MODE == M_SITES;  // column right of the tile
    constexpr int TL = TLIST;
    constexpr int BG4 = 4 * TSITES;  // offset of the background entry
    int *P = sm.P;
    auto &wl = sm.wl;
    int &nb_s = sm.nb_s;
    int *act_w = sm.act_w;
    const int W = a.g.W, H = a.g.H;
    const int tx = lt % a.g.ntx, ty = lt / a.g.ntx;
    const int gx0 = tx * TW, gy0 = ty * TH;
    const int tw = min(TW, W - gx0), th = min(TH, H - gy0);
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int lx0 = 2 * lane, lx1 = lx0 + 1, x4 = 4 * lx0;
    const bool v0 = lx0 < tw, v1 = lx1 < tw;
    const int hx = (gx0 + tw == W) ? 0 : gx0 + tw;  // column right of the tile
    const bool right_is_wrap = (gx0 + tw == W);
    const bool bottom_is_wrap = (gy0 + th == H);
    const int ly0 = wave * RPW;
    const int nr = max(0, min(RPW, th - ly0));  // tile rows owned by this wave
    uint16_t *mylist = wl[wave];
    // Unite the n contacts of the wave's list (contact c joins slots c and
    // c + TW; the list holds their byte offsets).  Lane L takes contacts L, L+64, ...; a lane whose union is done
    // takes its next contact at once, so one deep union does not hold up the
    // other lanes of its round.
    auto unite_list = [&](int n) {
        wave_lds_fence();
        int i = lane, a = 0, b = 0;
        if (i < n) {
            const int c = mylist[i];  // byte offset of the upper site
            a = lds_ld(lds_entry(P, c));
            b = lds_ld(lds_entry(P, c + 4 * TW));
        }
        while (i < n) {
            int done;
            unite_step(P, a, b, done);
            if (done) {
                i += 64;
                if (i < n) {
                    const int c = mylist[i];
                    a = lds_ld(lds_entry(P, c));
                    b = lds_ld(lds_entry(P, c + 4 * TW));
                }
            }
        }
        wave_lds_fence();
    };
    // lane masks of the sites inside the tile, and of its last column
    const uint64_t in0 = ~0ull >> (64 - ((tw + 1) >> 1)), in1 = in0 >> (tw & 1);
    const uint64_t L0 = EVENW ? 0ull : in0 & ~in1, L1 = in1 & ~(in0 >> 1);

    if (threadIdx.x == 0) {  // first used after the barrier closing phase A
        nb_s = 0;
        P[TSITES] = final_entry(CODE_BG);
    }

    // ---- A0: issue every load of the wave's rows (and the row below) up front,
    // branch-free within the wave: invalid lanes read a clamped valid address.
    // pr[r] holds the bytes of sites lx0 (bits 0-7) and lx1 (bits 8 up).
    const int col = gx0 + (v0 ? lx0 : 0);
    uint32_t pr[RPW + 1];
    uint32_t hl[RPW];
#pragma unroll
    for (int r = 0; r <= RPW; ++r) {
        pr[r] = 0;
        if (r < RPW) hl[r] = 0;
        if (nr > 0 && (r < nr || (NEED_DOWN && r == nr))) {
            int gy = gy0 + ly0 + r;
            if (gy == H) gy = 0;  // ly0 + r <= th, so at most one wrap
            const uint8_t *row = a.in + static_cast<int64_t>(gy) * W;
            if constexpr (EVENW) {
                pr[r] = *reinterpret_cast<const uint16_t *>(row + col);
            } else {
                pr[r] = static_cast<uint32_t>(row[col]) | (static_cast<uint32_t>(row[col + (v1 ? 1 : 0)]) << 8);
            }
            if (NEED_HALO && r < nr) hl[r] = row[hx];  // same byte for every lane
        }
    }
    if (tw < TW) {
        // Sites past a ragged edge have no bonds: spins that differ from each
        // other, from every byte on their right and from the row below
        // (pr[r] bits 8 up exceed a byte); bond bytes and pixels 0.
#pragma unroll
        for (int r = 0; r <= RPW; ++r) {
            const uint32_t no0 = MODE == M_SW ? (r & 1) : 0u, no1 = MODE == M_SW ? (0x102u + (r & 1)) << 8 : 0u;
            pr[r] = v1 ? pr[r] : (v0 ? pr[r] & 0xFFu : no0) | no1;
        }
    }
    if constexpr (MODE == M_SITES) {  // an open boundary: nothing below the last row
        if (bottom_is_wrap) {
#pragma unroll
            for (int r = 1; r <= RPW; ++r)
                if (ly0 + r == th) pr[r] = 0;
        }
    }

    // ---- A1: bonds as lane masks, then row by row the sites' labels: a run
    // takes the label of one run above it (one of its contacts), or its own
    // start without a contact.  Most contacts are the only one of their run
    // (at a critical point about 50 of a row's 128 sites have one, about 10
    // are left to unite), so this leaves a fifth of the unions, each four
    // dependent LDS reads and an atomic a step, and as few entries to
    // compress: a labeled run start already points at its label.  Sweep of
    // the q = 3 lattice 16384^2, every contact united -> labels passed down:
    // 1.173 -> 1.026 ms; labeling of 16384^2 random bonds 1.251 -> 1.061 ms.
    // The labels stay in registers: the code pass reads one entry a site and
    // packs it with a shift (codes are entries without their two low bits),
    // and no table of run masks, label masks or occupied sites is kept in LDS.
    // The kernel is bound by VALU issue (busy 0.95), so instructions count:
    // with that and the masks of ragged edges folded into the loaded bytes,
    // 185 VALU and 150 SALU a row became 143 and 111, and the same sweep
    // 1.026 -> 0.867 ms, the labeling 1.061 -> 0.930 ms.
    uint32_t xr = 0;
    int nact = 0;  // at most 2 * TSITES
    int ncon = 0;
    int lab0[RPW], lab1[RPW];  // labels of the lane's sites (byte offsets), BG4 for background
    EO prevD = EO{0ull, 0ull};
#pragma unroll
    for (int r = 0; r < RPW; ++r) lab0[r] = lab1[r] = BG4;
    // Odd W: lane r holds the block after row r's last pair, which only the last
    // lane of a row that starts on an odd site needs: one block for all rows
    // of the wave instead of a second one for each such row (q = 3 sweep of
    // 4097 x 4096 93.9 -> 91.7 us, 8191 x 8192 251 -> 244).
    U4 tail{};
    if constexpr (MODE == M_SW && !EVENW) {
        const uint32_t i_last = static_cast<uint32_t>(gy0 + ly0 + lane % RPW) * static_cast<uint32_t>(W) +
                                static_cast<uint32_t>(gx0 + TW - 1);
        tail = philox4x32_10(i_last >> 1, a.t, TAG_BOND, a.sid, __builtin_amdgcn_readfirstlane(a.k0),
                             __builtin_amdgcn_readfirstlane(a.k1));
    }
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        if (r >= nr) break;
        const int ly = ly0 + r;
        const int gy = gy0 + ly;
        const uint32_t cur = pr[r], dn = pr[r + 1];
        uint64_t mR0, mR1, mD0, mD1, O0 = ~0ull, O1 = ~0ull;
        uint64_t cross;  // the last column's right bond, which leaves the tile

        if constexpr (MODE == M_SW) {
            const uint32_t s0 = cur & 0xFFu, s1 = cur >> 8;
            const uint32_t d0 = dn & 0xFFu, d1 = dn >> 8;
            const uint32_t nxt = from_next_lane(s0);
            const uint32_t sr0 = (!EVENW && lane_bit(L0, lane)) ? hl[r] : s1;
            const uint32_t sr1 = lane_bit(L1, lane) ? hl[r] : nxt;
            const uint32_t i0 = static_cast<uint32_t>(gy) * static_cast<uint32_t>(W) + static_cast<uint32_t>(gx0 + lx0);
            uint32_t r0R, r0D, r1R, r1D;
            // the key schedule is recomputed per row (scalar adds) rather than
            // held in 20 scalar registers across the unrolled row loop
            uint32_t k0 = __builtin_amdgcn_readfirstlane(a.k0), k1 = __builtin_amdgcn_readfirstlane(a.k1);
            asm volatile("" : "+s"(k0), "+s"(k1));
            U4 blk;
            if constexpr (RKEYS) {
                blk = philox4x32_10_rk(i0 >> 1, a.t, TAG_BOND, a.sid, kernel_tile_args()->rk);
            } else {
                blk = philox4x32_10(i0 >> 1, a.t, TAG_BOND, a.sid, k0, k1);
            }
            if (EVENW || ((gy * W + gx0) & 1) == 0) {  // the pair (i0, i0+1) shares one block
                r0R = blk.v0;
                r0D = blk.v1;
                r1R = blk.v2;
                r1D = blk.v3;
            } else {
                // odd row start (odd W): i0 is the second site of its block,
                // i0 + 1 the first of the next lane's (the last lane's: tail)
                r0R = blk.v2;
                r0D = blk.v3;
                r1R = from_next_lane_or(blk.v0, __builtin_amdgcn_readlane(static_cast<int>(tail.v0), r));
                r1D = from_next_lane_or(blk.v1, __builtin_amdgcn_readlane(static_cast<int>(tail.v1), r));
            }
            // uniform flags are re-read per row (held across rows as lane
            // masks, they would spill)
            uint32_t tany = __builtin_amdgcn_readfirstlane(a.tany);
            uint8_t *bonds_out = uniform_ptr(a.bonds_out);
            asm volatile("" : "+s"(tany), "+s"(bonds_out));
            mR0 = lanes_eq(s0, sr0) & lanes_le(r0R, a.tm1);
            mD0 = lanes_eq(s0, d0) & lanes_le(r0D, a.tm1);
            mR1 = lanes_eq(s1, sr1) & lanes_le(r1R, a.tm1);
            mD1 = lanes_eq(s1, d1) & lanes_le(r1D, a.tm1);
            if (!tany) mR0 = mR1 = mD0 = mD1 = 0ull;
            if (bonds_out) {
                const uint32_t b0 = lane_bit(mR0, lane) | (lane_bit(mD0, lane) << 1);
                const uint32_t b1 = lane_bit(mR1, lane) | (lane_bit(mD1, lane) << 1);
                if (v1 && (EVENW || !(i0 & 1))) {
                    *reinterpret_cast<uint16_t *>(bonds_out + i0) = static_cast<uint16_t>(b0 | (b1 << 8));
                } else {
                    if (v0) bonds_out[i0] = static_cast<uint8_t>(b0);
                    if (v1) bonds_out[i0 + 1] = static_cast<uint8_t>(b1);
                }
            }
            nact += __popcll(mR0) + __popcll(mD0) + __popcll(mR1) + __popcll(mD1);  // 32-bit sums
            cross = (mR0 & L0) | (mR1 & L1);
        } else if constexpr (MODE == M_BONDS_PERIODIC || MODE == M_BONDS_OPEN) {
            mR0 = lanes_ne(cur & 0x001u, 0u);
            mD0 = lanes_ne(cur & 0x002u, 0u);
            mR1 = lanes_ne(cur & 0x100u, 0u);
            mD1 = lanes_ne(cur & 0x200u, 0u);
            cross = (mR0 & L0) | (mR1 & L1);
        } else {  // M_SITES: 4-connected occupied pixels, open boundary
            O0 = lanes_ne(cur & 0x00FFu, 0u);
            O1 = lanes_ne(cur & 0xFF00u, 0u);
            mD0 = O0 & lanes_ne(dn & 0x00FFu, 0u);
            mD1 = O1 & lanes_ne(dn & 0xFF00u, 0u);
            mR0 = O0 & O1;         // the last column's right neighbour reads 0 here
            mR1 = O1 & (O0 >> 1);
            cross = lanes_ne(hl[r], 0u) & ((O0 & L0) | (O1 & L1));
        }

        // Crossing bonds leave the tile: the last column's right bond here,
        // the last row's down bonds below.  They are merged by k_merge.
        xr |= cross ? 1u << r : 0u;
        const EO R = EO{mR0 & ~L0, mR1 & ~L1};
        const int base = ly * TW;
        // Run starts: site 2L starts a run unless bond 2L-1 -> 2L is present,
        // site 2L+1 unless bond 2L -> 2L+1 is; the run start of 2L is the last
        // start at or before it (a max-scan over the lanes below), in byte
        // offsets within the row (x4 = 4 lx0); lane 0's even site always
        // starts a run, at offset 0.
        const bool e_start = lane_bit(~(R.o << 1), lane);
        const bool o_start = lane_bit(~R.e, lane);
        const int below4 = wave_max_below(o_start ? x4 + 4 : (e_start ? x4 : 0));
        const int rs0 = e_start ? x4 : below4;
        const int rs1 = o_start ? x4 + 4 : rs0;
        int n0 = 4 * base + rs0, n1 = 4 * base + rs1;
        if constexpr (MODE == M_SITES) {
            n0 = lane_bit(O0, lane) ? n0 : BG4;
            n1 = lane_bit(O1, lane) ? n1 : BG4;
        }
        *reinterpret_cast<int2 *>(&P[base + lx0]) = make_int2(n0, n1);
        if (r > 0) {
            // every contact offers its upper site's label to the lower run's
            // start (one wave's LDS operations run in order; whichever offer
            // lands last stands); a contact whose label lost needs a union
            const int up0 = lab0[r > 0 ? r - 1 : 0], up1 = lab1[r > 0 ? r - 1 : 0];
            wave_lds_fence();
            if (lane_bit(prevD.e, lane)) lds_st(lds_entry(P, n0), up0);
            if (lane_bit(prevD.o, lane)) lds_st(lds_entry(P, n1), up1);
            wave_lds_fence();
            // (the background entry reads as itself: background keeps BG4)
            const int q0 = lds_ld(lds_entry(P, n0)), q1 = lds_ld(lds_entry(P, n1));
            n0 = MODE == M_SITES && n0 == BG4 ? BG4 : q0;
            n1 = MODE == M_SITES && n1 == BG4 ? BG4 : q1;
            *reinterpret_cast<int2 *>(&P[base + lx0]) = make_int2(n0, n1);
            const EO lost = EO{lanes_ne(static_cast<uint32_t>(n0), static_cast<uint32_t>(up0)) & prevD.e,
                               lanes_ne(static_cast<uint32_t>(n1), static_cast<uint32_t>(up1)) & prevD.o};
            // a full list is united at once (only rows this wave has
            // initialised are involved)
            if (ncon > TL - TW) {
                unite_list(ncon);
                ncon = 0;
            }
            const int up_own = 4 * (base - TW) + x4;  // the upper even site
            eo_append(mylist, ncon, lost, up_own, up_own + 4);
        }
        lab0[r] = n0;
        lab1[r] = n1;
        prevD = EO{mD0, mD1};
    }
    if (MODE == M_BONDS_OPEN || MODE == M_SITES) xr = right_is_wrap ? 0u : xr;
    if (lane == 0) {
        sm.xr_w[wave] = xr;
        act_w[wave] = nact;
        // the last tile row's down bonds cross the tile
        if (nr > 0 && ly0 + nr == th)
            sm.xd_s = MODE == M_BONDS_OPEN && bottom_is_wrap ? EO{0ull, 0ull} : prevD;
    }
    if (tw < TW) {  // sites past a ragged edge get background codes
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            lab0[r] = v0 ? lab0[r] : BG4;
            lab1[r] = v1 ? lab1[r] : BG4;
        }
    }
    __syncthreads();

    // ---- B: contacts with the next wave's first row, then all unions.  A
    // lower label that is still a root of that row on is linked below the
    // upper label by one compare-and-swap (upper labels lie above the row, so
    // a parent stays below its child); the contacts left are united.
    if (nr > 0 && ly0 + nr < th) {
        if (ncon > TL - TW) {
            unite_list(ncon);
            ncon = 0;
        }
        const int row4 = 4 * (ly0 + nr) * TW;
        const int up0 = nr == RPW ? lab0[RPW - 1] : 0, up1 = nr == RPW ? lab1[RPW - 1] : 0;
        const int2 low = make_int2(lds_ld(&P[(row4 >> 2) + lx0]), lds_ld(&P[(row4 >> 2) + lx0 + 1]));
        int got0 = -1, got1 = -1;
        if (lane_bit(prevD.e, lane) && low.x >= row4) got0 = link_root(P, low.x, up0);
        if (lane_bit(prevD.o, lane) && low.y >= row4) got1 = link_root(P, low.y, up1);
        const EO met = EO{lanes_eq(static_cast<uint32_t>(got0), static_cast<uint32_t>(low.x)) |
                              lanes_eq(static_cast<uint32_t>(got0), static_cast<uint32_t>(up0)),
                          lanes_eq(static_cast<uint32_t>(got1), static_cast<uint32_t>(low.y)) |
                              lanes_eq(static_cast<uint32_t>(got1), static_cast<uint32_t>(up1))};
        eo_append(mylist, ncon, eo_andnot(prevD, met), row4 - 4 * TW + x4, row4 - 4 * TW + x4 + 4);
    }
    unite_list(ncon);
    __syncthreads();

    // ---- C: the clusters that touch the tile border are claimed (one
    // thread per border position), then, after a barrier, every linked label
    // gets its cluster's final entry: the claimed root's, or that of the
    // unclaimed root's slot.  Lane L walks labels L, L+64, ... of the wave's
    // list up to the first entry that is negative (a claimed root, or a label
    // another lane has finished: either way the cluster's code) or its own (an
    // unclaimed root); a lane whose walk is done takes its next label at once.
    // Only linked labels (entry neither their own nor negative) are listed.
    auto compress_list = [&](int n) {
        wave_lds_fence();
        int i = lane, s0 = 0, x = 0;
        if (i < n) s0 = x = mylist[i];
        while (i < n) {
            const int p = lds_ld(lds_entry(P, x));
            if (p >= 0 && p != x) {
                x = p;
            } else {
                lds_st(lds_entry(P, s0), p | static_cast<int>(0x80000000u));
                i += 64;
                if (i < n) s0 = x = mylist[i];
            }
        }
        wave_lds_fence();
    };
    int32_t *gkey = a.gkey, *gparent = a.gparent, *gsize = a.gsize;
    if constexpr (KARG) {
        KernTileArgs *ka = kernel_tile_args();
        gkey = ka->gkey;
        gparent = ka->gparent;
        gsize = ka->gsize;
    }
    for (int t = threadIdx.x; t < EDGE; t += NT) {
        const int slot = border_slot<TH>(t, tw, th);
        if (slot < 0) continue;
        const int root4 = lroot(P, 4 * slot), root = root4 >> 2;
        int expect = root4;
        // (background ends at its own entry, which no claim matches)
        if (__hip_atomic_compare_exchange_strong(lds_entry(P, root4), &expect, CLAIMING, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
            const int k = atomicAdd(&nb_s, 1);
            lds_st(lds_entry(P, root4), final_entry(static_cast<uint32_t>(TSITES + k)));
            const int id = tile * CAP + k;
            gkey[id] = (gy0 + (root >> 7)) * W + gx0 + (root & (TW - 1));
            gparent[id] = id;
            if (gsize) gsize[id] = 0;
        }
    }
    __syncthreads();
    int nrs = 0;
    // The entries of the wave's sites are read up front (the loads overlap);
    // a flush of the list only rewrites linked labels of this wave.
    int2 ppr[RPW];
#pragma unroll
    for (int r = 0; r < RPW; ++r)
        ppr[r] = r < nr ? *reinterpret_cast<const int2 *>(&P[(ly0 + r) * TW + lx0]) : make_int2(0, 0);
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        if (r >= nr) break;
        if (nrs > TL - TW) {
            compress_list(nrs);
            nrs = 0;
        }
        // a label site whose entry is an offset below its own (a final entry
        // is negative, above every offset as an unsigned number)
        const uint32_t own = static_cast<uint32_t>(4 * (ly0 + r) * TW + x4);
        const EO linked = EO{lanes_eq(static_cast<uint32_t>(lab0[r]), own) & lanes_lt(static_cast<uint32_t>(ppr[r].x), own),
                             lanes_eq(static_cast<uint32_t>(lab1[r]), own + 4) &
                                 lanes_lt(static_cast<uint32_t>(ppr[r].y), own + 4)};
        eo_append(mylist, nrs, linked, static_cast<int>(own), static_cast<int>(own + 4));
    }
    compress_list(nrs);
    __syncthreads();

    // ---- E: per-site codes (the entry of the site's label), edge ids,
    // crossing bits.
    uint16_t *codes = a.codes, *edges = a.edges;
    uint64_t *xbits = a.xbits;
    int32_t *nbp = a.nb, *tile_act = a.tile_act;
    if constexpr (KARG) {
        KernTileArgs *ka = kernel_tile_args();
        codes = ka->codes;
        edges = ka->edges;
        xbits = ka->xbits;
        nbp = ka->nb;
        tile_act = ka->tile_act;
    }
    uint32_t *codes32 = reinterpret_cast<uint32_t *>(codes + static_cast<int64_t>(tile) * TSITES) +
                        ly0 * (TW / 2) + lane;
    // unrolled: the rows' lookups are independent, so their LDS loads overlap
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        if (r >= nr) break;
        const uint32_t code0 = entry_code(lds_ld(lds_entry(P, lab0[r])));
        const uint32_t code1 = entry_code(lds_ld(lds_entry(P, lab1[r])));
        codes32[r * (TW / 2)] = code0 | (code1 << 16);
    }
    uint16_t *edg = edges + static_cast<int64_t>(tile) * EDGE;
    for (int t = threadIdx.x; t < EDGE; t += NT) {
        const int slot = border_slot<TH>(t, tw, th);
        uint16_t eid = ID_NONE;
        if (slot >= 0) {
            int e = P[slot];  // a claimed root or coded label, or the site's label
            if (e >= 0) e = *lds_entry(P, e);
            eid = static_cast<uint16_t>(entry_code(e) - TSITES);  // a boundary id; background ends up past CAP
        }
        edg[t] = eid;
    }
    if (threadIdx.x == 0) {
        uint64_t *xb = xbits + static_cast<int64_t>(tile) * XW;
        int act = 0;
#pragma unroll
        for (int j = 0; j < XR; ++j) {
            unsigned long long xrt = 0;  // rows 64 j ... 64 j + 63: the waves (64 / RPW of them) holding them
            for (int w = j * (64 / RPW); w < min(NWAVE, (j + 1) * (64 / RPW)); ++w)
                xrt |= static_cast<unsigned long long>(sm.xr_w[w]) << ((w * RPW) & 63);
            xb[j] = xrt;
        }
        for (int w = 0; w < NWAVE; ++w) act += act_w[w];
        xb[XR] = sm.xd_s.e;      // bottom crossing bonds of even columns
        xb[XR + 1] = sm.xd_s.o;  // ... and of odd columns
        nbp[tile] = nb_s;
        if (MODE == M_SW && tile_act) tile_act[tile] = act;
    }
}

// 8 waves per SIMD (four 128 x 64 workgroups of eight waves per CU, or two of
// sixteen): the LDS leaves room for them and the registers are held to what 8
// waves allow (some scalar registers spill to vector lanes; the extra latency
// hiding is worth more).
// RPW_ = RPW_SMALL: twice the waves with half the rows each, for lattices of few
// tiles (see the launch).
constexpr int RPW_SMALL = 4;
template <int MODE, bool EVENW, bool BATCH, int TH_, int RPW_ = RPW>
__global__ __launch_bounds__(64 * TH_ / RPW_) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_tile(TileArgs a)
{
    static_assert(tile_fits<MODE, TH_, RPW_>, "8 waves per SIMD");
    __shared__ TileSmem<MODE, TH_, RPW_> sm;
    int tile, lt;  // tile in the arrays, tile inside its lattice
    if constexpr (BATCH) {
        tile = a.b.tile_base + xcd_remap(blockIdx.x, a.b.ntiles);
        load_batch_tile(a, tile, lt);
    } else {
        tile = lt = xcd_remap(blockIdx.x, a.g.ntiles);
        if (a.g.rev) tile = lt = a.g.ntiles - 1 - tile;
    }
    tile_body<MODE, EVENW, TH_, true, !BATCH && MODE == M_SW, RPW_>(a, tile, lt, sm);
}

// ---------------------------------------------------------------- merge ----

struct MergeArgs {
    Grid g;
    const uint16_t *edges;
    const uint64_t *xbits;
    const int32_t *gkey;
    int32_t *gparent;
    Batch b;                  // batched launches only
};

// Tile consolidation in passes of 64 crossing bonds: a tile's right edge (TH
// rows, 64 a pass) and its bottom edge (TW columns, two passes); a lane takes
// one crossing bond of a pass, and consecutive bonds that join the same pair of
// boundary ids are skipped.  A wave takes all passes of a tile or, on lattices
// whose passes fit the chip at once, one of them (see the launch): what bounds
// a pass is its chain of dependent global accesses (edge ids, then parents and
// keys, then swaps).  The workgroup size (blockDim, in waves) is the merge
// schedule's free parameter.
template <int TH_>
struct MergePasses {
    static constexpr int RIGHT = (TH_ + 63) / 64, N = RIGHT + 2;
};

// Passes pass0 .. pass0 + PASSES - 1 of one tile by the calling wave (`tile`
// indexes the tile arrays).
template <bool BATCH, int TH_, int PASSES>
__device__ __forceinline__ void merge_tile(MergeArgs a, const int tile, const int pass0)
{
    using S = Tile<TH_>;
    constexpr int TH = S::TH, CAP = S::CAP, EDGE = S::EDGE, XR = S::XR, XW = S::XW, RIGHT = MergePasses<TH_>::RIGHT;
    const int lane = threadIdx.x & 63;
    int tile0 = 0;  // first tile of the lattice in the arrays
    if constexpr (BATCH) {
        const LatticeDesc &L = a.b.lat[a.b.lat_of_tile[tile]];
        a.g = L.g;
        tile0 = L.tile0;
    }
    const int lt = tile - tile0;
    const int tx = lt % a.g.ntx, ty = lt / a.g.ntx;
    const int tw = min(TW, a.g.W - tx * TW), th = min(TH, a.g.H - ty * TH);
    const int ntR = tile0 + ty * a.g.ntx + (tx + 1 == a.g.ntx ? 0 : tx + 1);
    const int ntD = tile0 + (ty + 1 == a.g.nty ? 0 : ty + 1) * a.g.ntx + tx;
    const uint16_t *e = a.edges + static_cast<int64_t>(tile) * EDGE;
    const uint16_t *eR = a.edges + static_cast<int64_t>(ntR) * EDGE, *eD = a.edges + static_cast<int64_t>(ntD) * EDGE;
    const uint64_t *xb = a.xbits + static_cast<int64_t>(tile) * XW;
    // Each pass's crossing bond c of the lane (a row of the right edge or a
    // column of the bottom edge): the ids on both sides of it and of the bond
    // before it (for skipping repeats), all loaded up front and inside the
    // arrays, and whether the two bonds are there.
    uint16_t ia[PASSES], ib[PASSES], pa[PASSES], pb[PASSES];
    bool on[PASSES], before[PASSES];
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        const int pass = pass0 + k;
        const bool right = pass < RIGHT;
        const int c = 64 * (right ? pass : pass - RIGHT) + lane;
        const uint16_t *ea = right ? e + 2 * TW + TH : e + TW, *eb = right ? eR + 2 * TW : eD;
        const int cl = min(c, (right ? TH : TW) - 1), cm = max(cl - 1, 0);
        ia[k] = ea[cl];
        ib[k] = eb[cl];
        pa[k] = ea[cm];
        pb[k] = eb[cm];
        // rows of the right edge in words of 64, the bottom edge's even
        // columns, then its odd ones
        auto bit_of = [&](int i) {
            const uint64_t w = right ? xb[i >> 6] : ((i & 1) ? xb[XR + 1] : xb[XR]);
            return ((w >> (right ? i & 63 : i >> 1)) & 1ull) != 0ull;
        };
        on[k] = c < (right ? th : tw) && bit_of(cl);
        before[k] = c > 0 && bit_of(cm);
    }
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        // Both ends of a crossing bond are border sites, whose codes are
        // boundary ids (< CAP); the bound keeps any other entry from
        // addressing memory outside the tiles' tables.
        if (on[k] && !(before[k] && pa[k] == ia[k] && pb[k] == ib[k]) && ia[k] < CAP && ib[k] < CAP)
            gunite(a.gparent, a.gkey, tile * CAP + ia[k], (pass0 + k < RIGHT ? ntR : ntD) * CAP + ib[k],
                   a.g.ntiles <= MERGE_FRESH_TILES);
    }
}

template <bool BATCH, int TH_, bool SPLIT>
__global__ __launch_bounds__(1024) void k_merge(MergeArgs a)
{
    constexpr int NP = MergePasses<TH_>::N;
    const int job = blockIdx.x * static_cast<int>(blockDim.x >> 6) + wave_id();
    int tile = SPLIT ? job / NP : job;
    const int pass = SPLIT ? job - tile * NP : 0;
    if constexpr (BATCH) {
        if (tile >= a.b.ntiles) return;
        tile += a.b.tile_base;
    } else {
        if (tile >= a.g.ntiles) return;
        if (a.g.rev) tile = a.g.ntiles - 1 - tile;
    }
    merge_tile<BATCH, TH_, SPLIT ? 1 : NP>(a, tile, pass);
}

// -------------------------------------------------------------- flatten ----

struct FlatArgs {
    Grid g;
    const uint16_t *codes;
    const int32_t *gkey;
    int32_t *gparent;
    const int32_t *nb;
    uint8_t *spins;           // M_SW: written
    int32_t *labels;          // canonical labels or nullptr
    int32_t *tile_ncl;        // [ntiles]: clusters whose canonical root lies in the tile
    // cluster sizes (nullptr when not requested)
    int32_t *gsize;           // [ntiles][CAP]
    int32_t *row_count;       // [H][ntx]: roots per (row, tile column)
    int32_t *rl_slot;         // [ntiles][TSITES]: root slots in raster order
    int32_t *rl_size;         // size, or -(root id + 1) for boundary clusters
    uint32_t q, k0, k1, t, sid;
    int ising;
    Batch b;                  // batched launches only
    // few-cluster flips (M_FEW)
    const uint32_t *sel;      // [ntiles][CAP]: == stamp at the root id of a seeded boundary cluster
    uint32_t *seedmap;        // [ntiles][TSITES / 32]: interior roots that hold a seed (cleared here)
    uint32_t stamp;           // this sweep's mark (t + 1)
    uint32_t tflip;           // a seeded cluster flips iff its FEW word is below this
    uint32_t *ticket;         // cleared for the observables that follow, or nullptr
};

// The seed of seed tile j (Sec. III, few-cluster variant): the lattice is cut
// into few_b x few_b seed tiles (narrower at the right and bottom edges), j in
// raster order, and each draws one of its own sites from the block
// (j, t, SEED, sid): x from word 0, y from word 1, each floor(w * extent / 2^32).
__device__ __forceinline__ void seed_site(int j, int W, int H, int B, int ntx, uint32_t t, uint32_t sid, uint32_t k0,
                                          uint32_t k1, int &x, int &y)
{
    const int tx = j % ntx, ty = j / ntx;
    const uint32_t bw = static_cast<uint32_t>(min(B, W - tx * B)), bh = static_cast<uint32_t>(min(B, H - ty * B));
    const U4 b = philox4x32_10(static_cast<uint32_t>(j), t, TAG_SEED, sid, k0, k1);
    x = tx * B + static_cast<int>((static_cast<uint64_t>(b.v0) * bw) >> 32);
    y = ty * B + static_cast<int>((static_cast<uint64_t>(b.v1) * bh) >> 32);
}

// Whether the seeded cluster with canonical root R flips (one draw per
// distinct cluster, Sec. III).
__device__ __forceinline__ bool few_flips(uint32_t R, const FlatArgs &a)
{
    const U4 b = philox4x32_10(R >> 2, a.t, TAG_FEW, a.sid, a.k0, a.k1);
    return pick(b, R & 3u) < a.tflip;
}

// Spin byte <-> state 0..q-1 (Ising bytes are -1 / +1 for states 0 / 1).
__device__ __forceinline__ uint32_t state_of_byte(uint32_t v, int ising) { return ising ? (v == 1u ? 1u : 0u) : v; }

// Clusters that hold a seed: one thread per seed tile finds the code of its
// seed's site.  A boundary cluster is marked at its root id with this sweep's
// stamp; an interior cluster by the bit of its root slot in its tile's seed
// map, which the flatten of that tile reads and clears.
struct SeedArgs {
    Grid g;
    const uint16_t *codes;
    const int32_t *gparent;
    uint32_t *sel;
    uint32_t *seedmap;
    uint32_t stamp, t, sid, k0, k1;
    int few_b, few_ntx, nseed;
};

template <int TH_>
__global__ __launch_bounds__(NT) void k_seed(SeedArgs a)
{
    using S = Tile<TH_>;
    const int j = static_cast<int>(blockIdx.x) * NT + static_cast<int>(threadIdx.x);
    if (j >= a.nseed) return;
    int x, y;
    seed_site(j, a.g.W, a.g.H, a.few_b, a.few_ntx, a.t, a.sid, a.k0, a.k1, x, y);
    const int lt = (y / S::TH) * a.g.ntx + x / TW;
    const int slot = (y % S::TH) * TW + x % TW;
    const uint32_t code = a.codes[static_cast<int64_t>(lt) * S::TSITES + slot];
    if (code >= static_cast<uint32_t>(S::TSITES)) {
        a.sel[gfind(a.gparent, lt * S::CAP + static_cast<int>(code) - S::TSITES)] = a.stamp;
    } else {
        const uint32_t root = code;
        atomicOr(&a.seedmap[static_cast<int64_t>(lt) * (S::TSITES / 32) + (root >> 5)], 1u << (root & 31u));
    }
}

// New spin byte of the cluster whose canonical root is R (Sec. II.D: one
// uniform draw per cluster, here taken at the minimum site index).
__device__ __forceinline__ uint8_t flip_byte(uint32_t R, const FlatArgs &a)
{
    const U4 b = philox4x32_10(R >> 2, a.t, TAG_FLIP, a.sid, a.k0, a.k1);
    const uint32_t st = draw_state(pick(b, R & 3u), a.q);
    return static_cast<uint8_t>(a.ising ? 2u * st - 1u : st);
}

constexpr int GSLOTS = 256;  // roots a tile adds its parts of up for

// LDS of the flatten phase.
template <int MODE, bool SIZES, int TH_, int RPW_ = RPW>
struct FlatSmem {
    static constexpr int TH = TH_, TSITES = TW * TH, CAP = 2 * (TW + TH), NWAVE = TH / RPW_;
    // new spin byte per code (root slot or TSITES + boundary id); M_FEW: new
    // state, FEW_KEEP = no change
    uint8_t ST[MODE == M_SW || MODE == M_FEW ? TSITES + CAP : 1];
    int32_t Rb[CAP];                              // canonical root (site index) per boundary id
    int32_t Gid[CAP];                             // root id per boundary id
    uint16_t rl[NWAVE][RPW_ * TW];                // interior roots of each wave's rows
    int ncl_w[NWAVE];
    int32_t Ci[SIZES ? TSITES : 1];               // sizes of interior clusters
    int32_t Cb[SIZES ? CAP : 1];                  // per-tile part of boundary clusters
    int32_t root_s[SIZES ? GSLOTS : 1];           // root id of a slot, -1 while free
    int32_t part_s[SIZES ? GSLOTS : 1];           // the tile's sites in that root's cluster
    int32_t rowc[TH];
    uint32_t seedw_s[MODE == M_FEW ? NWAVE : 1][RPW_ * TW / 32];  // M_FEW: seed-map words of each wave's rows
};

__device__ __forceinline__ void load_batch_flat(FlatArgs &a, int tile, int &lt)
{
    const LatticeDesc &L = a.b.lat[a.b.lat_of_tile[tile]];
    a.g = L.g;
    a.spins = L.spins;
    a.labels = L.labels;
    a.q = L.q;
    a.k0 = L.k0;
    a.k1 = L.k1;
    a.sid = L.sid;
    a.ising = L.ising;
    a.t = *a.b.t;
    lt = tile - L.tile0;
}

constexpr uint8_t FEW_KEEP = 0xFF;

// Exclusive prefix sums of v[0 .. n - 1] in place by one wave (n <= TH <= 128).
template <int TH>
__device__ __forceinline__ void exclusive_rows(int32_t *v, int n, int lane)
{
    uint32_t carry = 0;
#pragma unroll
    for (int y = 0; y < TH; y += 64) {
        const uint32_t x = y + lane < n ? static_cast<uint32_t>(v[y + lane]) : 0u;
        const uint32_t s = wave_scan_u32(x);
        if (y + lane < n) v[y + lane] = static_cast<int32_t>(carry + s - x);
        carry += __builtin_amdgcn_readlane(static_cast<int>(s), 63);
    }
}

// The flatten + flip of one tile (`tile` in the arrays, `lt` inside its
// lattice), by a Tile<TH>::NT-thread workgroup.  M_FEW flips only the seeded
// clusters whose draw says so and writes only their sites.
template <int MODE, bool SIZES, int TH_, int RPW_ = RPW>
__device__ __forceinline__ void flatten_body(FlatArgs a, const int tile, const int lt,
                                             FlatSmem<MODE, SIZES, TH_, RPW_> &sm)
{
    using S = Tile<TH_>;
    constexpr int TH = S::TH, TSITES = S::TSITES, CAP = S::CAP;
    constexpr int RPW = RPW_, NWAVE = TH / RPW, NT = 64 * NWAVE;  // rows per wave
    constexpr int BPT = (CAP + NT - 1) / NT;  // boundary ids per thread
    constexpr int NCODE = CAP + TSITES;
    uint8_t *ST = sm.ST;
    int32_t *Rb = sm.Rb, *Gid = sm.Gid;
    auto &rl = sm.rl;
    int *ncl_w = sm.ncl_w;
    int32_t *Ci = sm.Ci, *Cb = sm.Cb, *rowc = sm.rowc;
    const int W = a.g.W;
    const int tx = lt % a.g.ntx, ty = lt / a.g.ntx;
    const int gx0 = tx * TW, gy0 = ty * TH;
    const int tw = min(TW, W - gx0), th = min(TH, a.g.H - gy0);
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int lx0 = 2 * lane;
    const int ly0 = wave * RPW;
    const int nr = max(0, min(RPW, th - ly0));
    const int nbt = a.nb[tile];
    if (lt == 0 && threadIdx.x == 0 && a.ticket) *a.ticket = 0u;
    // each boundary id's parent and key (ids threadIdx.x + j NT), issued with
    // the count's loads (entries past nb are read, not used); a root's key is
    // its cluster's canonical label
    int broot[BPT], bR[BPT];
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
        const int k = static_cast<int>(threadIdx.x) + j * NT;
        broot[j] = bR[j] = 0;
        if (k < CAP) {
            broot[j] = a.gparent[tile * CAP + k];
            bR[j] = a.gkey[tile * CAP + k];
        }
    }

    if constexpr (SIZES) {
        // the scan's closing slot and the largest-size slot after the
        // per-(row, tile column) counts start at zero (no other block writes them)
        if (lt == 0 && threadIdx.x < 2) a.row_count[static_cast<int64_t>(a.g.H) * a.g.ntx + threadIdx.x] = 0;
        for (int k = threadIdx.x; k < TSITES; k += NT) Ci[k] = 0;
        for (int k = threadIdx.x; k < CAP; k += NT) Cb[k] = 0;
        for (int k = threadIdx.x; k < GSLOTS; k += NT) {
            sm.root_s[k] = -1;
            sm.part_s[k] = 0;
        }
    }
    // M_FEW: the seed-map words of this wave's rows (word l in lane l), cleared
    // for the next sweep
    constexpr int SEEDW = RPW * TW / 32;
    static_assert(GSLOTS == 256, "a slot is the top byte of a product");
    static_assert(SEEDW <= 64, "a seed-map word per lane");
    uint32_t seedw = 0;
    if constexpr (MODE == M_FEW) {
        if (lane < SEEDW) {
            uint32_t *w = a.seedmap + static_cast<int64_t>(tile) * (TSITES / 32) + ly0 * (TW / 32) + lane;
            seedw = *w;
            if (seedw) *w = 0u;
        }
    }
    uint32_t cc[RPW];
    const uint32_t *codes32 = reinterpret_cast<const uint32_t *>(a.codes + static_cast<int64_t>(tile) * TSITES);
#pragma unroll
    for (int r = 0; r < RPW; ++r) cc[r] = r < nr ? codes32[((ly0 + r) * TW + lx0) >> 1] : 0u;

    // interior roots (code = own slot) of the wave's rows, compacted
    int nroot = 0;
    uint16_t *mylist = rl[wave];
#pragma unroll
    for (int r = 0; r < RPW; ++r) {
        if (r >= nr) break;  // unrolled: cc[] stays indexed by constants
        const int base = (ly0 + r) * TW;
        const EO m = EO{lanes_eq(cc[r] & 0xFFFFu, static_cast<uint32_t>(base + lx0)),
                        lanes_eq(cc[r] >> 16, static_cast<uint32_t>(base + lx0 + 1))};
        eo_append(mylist, nroot, m, base + lx0, base + lx0 + 1);
    }
    wave_lds_fence();
    if constexpr (MODE == M_SW) {
        for (int i = lane; i < nroot; i += 64) {
            const int slot = mylist[i];
            ST[slot] = flip_byte(static_cast<uint32_t>((gy0 + (slot >> 7)) * W + gx0 + (slot & (TW - 1))), a);
        }
    } else if constexpr (MODE == M_FEW) {
        // a seeded interior cluster that flips takes the other state of its
        // root (every site of a cluster has the same spin); the interior roots
        // of the wave's list lie in its own rows, whose seed-map words the
        // wave keeps in its own LDS words; a seeded root's spin is loaded
        // ahead of the draw
        uint32_t *myseed = sm.seedw_s[wave];
        if (lane < SEEDW) myseed[lane] = seedw;
        wave_lds_fence();
        for (int i = lane; i < nroot; i += 64) {
            const int slot = mylist[i];
            const uint32_t R = static_cast<uint32_t>((gy0 + (slot >> 7)) * W + gx0 + (slot & (TW - 1)));
            const uint32_t word = myseed[(slot >> 5) - ly0 * (TW / 32)];
            const bool seeded = (word >> (slot & 31)) & 1u;
            uint32_t old = 0;
            if (seeded) old = a.spins[R];
            uint8_t v = FEW_KEEP;
            if (seeded && few_flips(R, a)) v = static_cast<uint8_t>(1u - state_of_byte(old, a.ising));
            ST[slot] = v;
        }
    }
    // boundary ids: the root and its key (the cluster's minimum site index),
    // loaded at the start
    int nbr = 0;
#pragma unroll
    for (int j = 0; j < BPT; ++j) {
        const int k = static_cast<int>(threadIdx.x) + j * NT;
        if (k < nbt) {
            const int id = tile * CAP + k;
            int r = broot[j], key = bR[j];
            uint32_t old = 0;
            if constexpr (MODE == M_FEW) old = a.spins[bR[j]];  // the id's own tile-local root, in this tile
            if (r != id) {  // below a root (the merge keeps trees shallow): walk up, take the root's key
                r = gfind(a.gparent, r);
                key = a.gkey[r];
            }
            Rb[k] = key;
            Gid[k] = r;
            nbr += r == id;
            if constexpr (MODE == M_SW) ST[TSITES + k] = flip_byte(static_cast<uint32_t>(key), a);
            if constexpr (MODE == M_FEW) {
                // seeded iff its root carries this sweep's mark; the old state
                // was read at the id's own tile-local root (a site of this
                // tile, not yet written)
                uint8_t v = FEW_KEEP;
                if (a.sel[r] == a.stamp && few_flips(static_cast<uint32_t>(key), a))
                    v = static_cast<uint8_t>(1u - state_of_byte(old, a.ising));
                ST[TSITES + k] = v;
            }
        }
    }
    {
        const unsigned long long s = wave_sum(static_cast<unsigned long long>(nbr));
        if (lane == 0) ncl_w[wave] = static_cast<int>(s) + nroot;
    }
    __syncthreads();
    if (threadIdx.x == 0 && a.tile_ncl) {
        int n = 0;
        for (int w = 0; w < NWAVE; ++w) n += ncl_w[w];
        a.tile_ncl[tile] = n;
    }

    // The lookups of all rows first, then the stores: a branch between the rows
    // would have each wait for its own LDS reads (16384^2, branches -> none: spins
    // 255 -> 249 us, labels of random bonds 383 -> 358).  `whole`: every row
    // starts on an even site and ends past the wave's last lane, so a lane's
    // pair is one store; otherwise rows that start on an odd site are stored
    // site by site.
    const bool v0 = lx0 < tw, v1 = lx0 + 1 < tw;
    const bool whole = tw == TW && (W & 1) == 0;
    auto first_of = [&](int r) { return static_cast<int64_t>(gy0 + ly0 + r) * W + gx0; };
    if constexpr (MODE == M_SW || MODE == M_FEW) {
        // (sites past a ragged tile edge carry CODE_BG: any entry is looked up,
        // none stored)
        uint32_t st0[RPW], st1[RPW];
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            st0[r] = ST[min(cc[r] & 0xFFFFu, static_cast<uint32_t>(NCODE - 1))];
            st1[r] = ST[min(cc[r] >> 16, static_cast<uint32_t>(NCODE - 1))];
        }
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            if (r >= nr) break;
            const int64_t row = first_of(r);
            uint8_t *out = a.spins + row;
            // only the sites of flipping clusters are written (M_FEW)
            const bool f0 = v0 && (MODE == M_SW || st0[r] != FEW_KEEP), f1 = v1 && (MODE == M_SW || st1[r] != FEW_KEEP);
            uint32_t b0 = st0[r], b1 = st1[r];
            if (MODE == M_FEW && a.ising) {
                b0 = (2u * b0 - 1u) & 0xFFu;
                b1 = (2u * b1 - 1u) & 0xFFu;
            }
            if (MODE == M_SW && whole) {
                *reinterpret_cast<uint16_t *>(out + lx0) = static_cast<uint16_t>(b0 | (b1 << 8));
            } else if (f0 && f1 && (row & 1) == 0) {
                *reinterpret_cast<uint16_t *>(out + lx0) = static_cast<uint16_t>(b0 | (b1 << 8));
            } else {
                if (f0) out[lx0] = static_cast<uint8_t>(b0);
                if (f1) out[lx0 + 1] = static_cast<uint8_t>(b1);
            }
        }
    }
    if (a.labels) {
        auto label_of = [&](uint32_t c) {  // straight-line: the table entry of a boundary id, else the root's site
            const int b = Rb[min(max(static_cast<int>(c) - TSITES, 0), CAP - 1)];
            const int own = (gy0 + static_cast<int>(c >> 7)) * W + gx0 + static_cast<int>(c & (TW - 1));
            const int v = c >= static_cast<uint32_t>(TSITES) ? b : own;
            return c == CODE_BG ? -1 : v;
        };
        int32_t R0[RPW], R1[RPW];
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            R0[r] = label_of(cc[r] & 0xFFFFu);
            R1[r] = label_of(cc[r] >> 16);
        }
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            if (r >= nr) break;
            const int64_t row = first_of(r);
            int32_t *out = a.labels + row;
            if (whole) {
                *reinterpret_cast<int2 *>(out + lx0) = make_int2(R0[r], R1[r]);
            } else if (v1 && (row & 1) == 0) {
                *reinterpret_cast<int2 *>(out + lx0) = make_int2(R0[r], R1[r]);
            } else {
                if (v0) out[lx0] = R0[r];
                if (v1) out[lx0 + 1] = R1[r];
            }
        }
    }
    if constexpr (SIZES) {
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            if (r >= nr) break;
            const uint32_t c0 = cc[r] & 0xFFFFu, c1 = cc[r] >> 16;
            if (v0 && c0 != CODE_BG) atomicAdd(c0 < static_cast<uint32_t>(TSITES) ? &Ci[c0] : &Cb[c0 - TSITES], 1);
            if (v1 && c1 != CODE_BG) atomicAdd(c1 < static_cast<uint32_t>(TSITES) ? &Ci[c1] : &Cb[c1 - TSITES], 1);
        }
    }

    if constexpr (SIZES) {
        __syncthreads();
        // boundary clusters: add this tile's part at the global root id.  Many
        // of a tile's ids belong to the same cluster (the spanning one above
        // all): their parts are added up in a small table first, so that its
        // root takes one atomic a tile (an id whose slot is another root's goes
        // to memory by itself).  4096^2, q = 3, sweep with its list, an atomic
        // an id -> this: 306 -> 190 us at 1.4 beta_c, 157.1 -> 156.5 at beta_c.
        auto give = [&](int root, int n) {
            __hip_atomic_fetch_add(&a.gsize[root], n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        for (int k = threadIdx.x; k < nbt; k += NT) {
            const int root = Gid[k], n = Cb[k];
            if (n == 0) continue;
            const int h = static_cast<int>((static_cast<uint32_t>(root) * 0x9E3779B1u) >> 24);
            const int was = atomicCAS(&sm.root_s[h], -1, root);
            if (was == -1 || was == root)
                atomicAdd(&sm.part_s[h], n);
            else
                give(root, n);
        }
        // canonical roots of this tile in raster order: per-row counts, then positions
        EO rm[RPW];
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            rm[r] = EO{0ull, 0ull};
            if (r >= nr) continue;
            const int ly = ly0 + r;
            const int base = ly * TW;
            bool isr[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int s = lx0 + j;
                const uint32_t code = (cc[r] >> (16 * j)) & 0xFFFFu;
                const int32_t self = (gy0 + ly) * W + gx0 + s;
                const int k = static_cast<int>(code) - TSITES;  // boundary id
                isr[j] = s < tw && code != CODE_BG &&
                         (code == static_cast<uint32_t>(base + s) ||
                          (k >= 0 && Gid[k] == tile * CAP + k && Rb[k] == self));
            }
            rm[r] = EO{__ballot(isr[0]), __ballot(isr[1])};
            if (lane == 0) {
                const int n = __popcll(rm[r].e) + __popcll(rm[r].o);
                rowc[ly] = n;
                a.row_count[static_cast<int64_t>(gy0 + ly) * a.g.ntx + tx] = n;
            }
        }
        __syncthreads();
        if (wave == 0) exclusive_rows<TH>(rowc, th, lane);
        for (int k = threadIdx.x; k < GSLOTS; k += NT)
            if (sm.part_s[k]) give(sm.root_s[k], sm.part_s[k]);
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RPW; ++r) {
            if (r >= nr) break;
            const int ly = ly0 + r;
            const int base = ly * TW;
            // ascending site order within the row: even sites below 2L+j, odd sites below
            const int below = lanes_below(rm[r].e) + lanes_below(rm[r].o);
            const int be = lane_bit(rm[r].e, lane) ? 1 : 0;
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                if (!lane_bit(j ? rm[r].o : rm[r].e, lane)) continue;
                const int s = lx0 + j;
                const int pos = rowc[ly] + below + (j ? be : 0);
                const uint32_t code = (cc[r] >> (16 * j)) & 0xFFFFu;
                const int64_t o = static_cast<int64_t>(tile) * TSITES + pos;
                a.rl_slot[o] = base + s;
                a.rl_size[o] = (code >= static_cast<uint32_t>(TSITES))
                                   ? -(tile * CAP + static_cast<int>(code) - TSITES + 1)
                                   : Ci[base + s];
            }
        }
    }
}

template <int MODE, bool SIZES, bool BATCH, int TH_, int RPW_ = RPW>
__global__ __launch_bounds__(64 * TH_ / RPW_) void k_flatten(FlatArgs a)
{
    __shared__ FlatSmem<MODE, SIZES, TH_, RPW_> sm;
    int tile, lt;  // tile in the arrays, tile inside its lattice
    if constexpr (BATCH) {
        tile = a.b.tile_base + xcd_remap(blockIdx.x, a.b.ntiles);
        load_batch_flat(a, tile, lt);
    } else {
        tile = lt = xcd_remap(blockIdx.x, a.g.ntiles);
        if (a.g.rev) tile = lt = a.g.ntiles - 1 - tile;
    }
    flatten_body<MODE, SIZES, TH_, RPW_>(a, tile, lt, sm);
}

// Sum of n per-tile int32 counters (256-byte aligned) by one workgroup.
__global__ __launch_bounds__(1024) void k_sum_tiles(const int32_t *v, int n, int32_t *out) { sum_tiles(v, n, out); }

// ------------------------------------------------------------ root list ----

// Exclusive scan of n int32 values in blocks of SCAN_ITEMS; block totals go to
// `totals` (scanned by the next level).
constexpr int SCAN_ITEMS = NT * 8;

__global__ __launch_bounds__(NT) void k_scan_block(const int32_t *in, int32_t *out, int64_t n, int32_t *totals)
{
    __shared__ uint32_t part[NWAVE];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * SCAN_ITEMS + threadIdx.x * 8;
    uint32_t v[8], sum = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        v[j] = (base + j < n) ? static_cast<uint32_t>(in[base + j]) : 0u;
        sum += v[j];
    }
    const uint32_t s = wave_scan_u32(sum);
    const int w = wave_id();
    if ((threadIdx.x & 63) == 63) part[w] = s;
    __syncthreads();
    uint32_t acc = s - sum, all = 0;
#pragma unroll
    for (int j = 0; j < NWAVE; ++j) {
        acc += j < w ? part[j] : 0u;
        all += part[j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (base + j < n) out[base + j] = static_cast<int32_t>(acc);
        acc += v[j];
    }
    if (threadIdx.x == 0 && totals) totals[blockIdx.x] = static_cast<int32_t>(all);
}

__global__ __launch_bounds__(NT) void k_scan_add(int32_t *out, int64_t n, const int32_t *offs)
{
    const int64_t i = static_cast<int64_t>(blockIdx.x) * NT + threadIdx.x;
    if (i < n) out[i] += offs[i / SCAN_ITEMS];
}

struct EmitArgs {
    Grid g;
    const int32_t *row_count; // [H*ntx] roots per (row, tile column) (DIRECT)
    const int32_t *row_off;   // [H*ntx + 1] their exclusive scan inside blocks of SCAN_ITEMS (otherwise)
    const int32_t *block_off; // offsets of the blocks, or nullptr if there is one
    const int32_t *rl_slot;
    const int32_t *rl_size;
    const int32_t *gsize;
    int32_t *roots;
    int32_t *sizes;
    int32_t *max_size;        // largest size (atomic max), or nullptr
    int32_t *n_clusters;      // the number of clusters (the offsets' total), or nullptr
    int32_t *n_host;          // the same, in host memory, or nullptr
};

// Write each tile's roots (ascending site index within a row) at their global
// positions; boundary clusters take their size from the global root id.
// DIRECT: a tile adds up itself the counts that come before its rows' roots
// (every count of the rows above it, then its own rows' up to its column);
// the counts are few enough that reading them again in every tile is cheaper
// than the scan's launches.
// Bound by latency on small lattices.  With the rows' counts added up one after
// the other by one thread (here and in the flatten), a three-launch scan and an
// atomic on the largest size from every wave, a sweep with sizes took 58 us on
// 512 x 500 (q = 3), now 44; 352 -> 159 on 4096^2 and 4726 -> 1909 on 16384^2
// (there the atomics).
template <int TH_, bool DIRECT>
__device__ __forceinline__ void emit_body(const EmitArgs &a, const int tile)
{
    constexpr int TH = Tile<TH_>::TH, TSITES = Tile<TH_>::TSITES, RW = (TH + NWAVE - 1) / NWAVE;
    __shared__ int32_t rstart[TH];  // roots of the tile in the rows above
    __shared__ int32_t rfirst[TH];  // global position of the row's first root in the tile
    __shared__ int32_t rsum[DIRECT ? TH : 1];
    __shared__ uint32_t red[NWAVE];
    __shared__ int32_t n_s, mx_s;
    const int ntx = a.g.ntx, tx = tile % ntx, ty = tile / ntx;
    const int gx0 = tx * TW, gy0 = ty * TH;
    const int th = min(TH, a.g.H - gy0);
    const int lane = threadIdx.x & 63, w = wave_id();
    // the thread's first entry, read ahead of its use (inside the tile's list,
    // whatever it holds)
    const int64_t list = static_cast<int64_t>(tile) * TSITES;
    int slot = a.rl_slot[list + threadIdx.x], sz = a.rl_size[list + threadIdx.x];
    if (threadIdx.x == 0) mx_s = 0;
    if constexpr (DIRECT) {
        uint32_t above = 0;
        for (int i = threadIdx.x; i < gy0 * ntx; i += NT) above += static_cast<uint32_t>(a.row_count[i]);
        uint32_t v[RW];  // the wave's rows w, w + NWAVE, ...: all loads first
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const int ly = w + r * NWAVE;
            v[r] = ly < th && lane < ntx ? static_cast<uint32_t>(a.row_count[(gy0 + ly) * ntx + lane]) : 0u;
        }
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const int ly = w + r * NWAVE;
            if (ly >= th) break;
            uint32_t all = v[r], left = lane < tx ? v[r] : 0u, own = lane == tx ? v[r] : 0u;
            for (int x = lane + 64; x < ntx; x += 64) {
                const uint32_t u = static_cast<uint32_t>(a.row_count[(gy0 + ly) * ntx + x]);
                all += u;
                left += x < tx ? u : 0u;
                own += x == tx ? u : 0u;
            }
            all = wave_sum_u32(all);
            left = wave_sum_u32(left);
            own = wave_sum_u32(own);
            if (lane == 0) {
                rsum[ly] = static_cast<int32_t>(all);
                rfirst[ly] = static_cast<int32_t>(left);
                rstart[ly] = static_cast<int32_t>(own);
            }
        }
        above = wave_sum_u32(above);
        if (lane == 0) red[w] = above;
    } else if (w == 0) {
        auto off = [&](int64_t i) { return a.row_off[i] + (a.block_off ? a.block_off[i / SCAN_ITEMS] : 0); };
        for (int ly = lane; ly < th; ly += 64) {
            const int64_t ix = static_cast<int64_t>(gy0 + ly) * ntx + tx;
            const int32_t first = off(ix);
            rfirst[ly] = first;
            rstart[ly] = off(ix + 1) - first;
        }
        if (a.n_clusters && tile == 0 && lane == 0) *a.n_clusters = off(static_cast<int64_t>(a.g.H) * ntx);
    }
    __syncthreads();
    if (w == 0) {
        uint32_t carry = 0, carry_sum = 0;
        if constexpr (DIRECT)
            for (int j = 0; j < NWAVE; ++j) carry_sum += red[j];
#pragma unroll
        for (int y = 0; y < TH; y += 64) {
            const bool in = y + lane < th;
            const uint32_t own = in ? static_cast<uint32_t>(rstart[y + lane]) : 0u, s = wave_scan_u32(own);
            if (in) rstart[y + lane] = static_cast<int32_t>(carry + s - own);
            carry += __builtin_amdgcn_readlane(static_cast<int>(s), 63);
            if constexpr (DIRECT) {
                const uint32_t all = in ? static_cast<uint32_t>(rsum[y + lane]) : 0u, t = wave_scan_u32(all);
                if (in) rfirst[y + lane] += static_cast<int32_t>(carry_sum + t - all);
                carry_sum += __builtin_amdgcn_readlane(static_cast<int>(t), 63);
            }
        }
        if (lane == 0) n_s = static_cast<int32_t>(carry);
        // the last band of rows ends with the number of clusters
        if (DIRECT && a.n_clusters && tile == a.g.ntiles - 1 && lane == 0) {
            *a.n_clusters = static_cast<int32_t>(carry_sum);
            if (a.n_host) *a.n_host = static_cast<int32_t>(carry_sum);
        }
    }
    __syncthreads();
    const int n = n_s;
    int mx = 0;
    for (int j = threadIdx.x; j < n; j += NT) {
        if (j >= NT) {
            slot = a.rl_slot[list + j];
            sz = a.rl_size[list + j];
        }
        const int ly = slot >> 7;
        const int pos = rfirst[ly] + (j - rstart[ly]);
        const int size = sz >= 0 ? sz : a.gsize[-sz - 1];
        a.roots[pos] = (gy0 + ly) * a.g.W + gx0 + (slot & (TW - 1));
        a.sizes[pos] = size;
        mx = max(mx, size);
    }
    if (a.max_size) {
        // one atomic a tile, and none from a tile whose largest is no larger
        // than what is there (a stale value is smaller still)
        if (mx > 0) atomicMax(&mx_s, mx);
        __syncthreads();
        if (threadIdx.x == 0 && mx_s > *a.max_size) atomicMax(a.max_size, mx_s);
    }
}

template <int TH_, bool DIRECT>
__global__ __launch_bounds__(NT) void k_emit(EmitArgs a)
{
    emit_body<TH_, DIRECT>(a, xcd_remap(blockIdx.x, a.g.ntiles));
}

// ------------------------------------------------------- small lattices ---
//
// A lattice of one tile (W <= SMALL_W, H <= SMALL_H) is swept entirely inside one
// workgroup: spins and union-find parents stay in LDS for all n sweeps of one
// launch, so a sweep costs neither launches nor an
// HBM round trip (a 64 x 64 lattice is launch-latency bound otherwise).  The
// bonds, canonical labels and new states are those of the tiled path; every
// bond, wrap bonds included, is a union inside the workgroup.

// Per-sweep record of sw_sweep_history: active bonds, clusters, largest cluster
// (-1: not measured), satisfied bonds and state counts of the new spins.
enum { HIST_ACTIVE = 0, HIST_NCLUST = 1, HIST_MAXCL = 2, HIST_NSAT = 3, HIST_COUNTS = 4, HIST_LEN = 12 };

struct SmallArgs {
    int W, H;
    uint8_t *spins;       // read at the start, written at the end
    uint8_t *bonds_out;   // packed bonds of the last sweep, or nullptr
    int32_t *labels;      // canonical labels of the last sweep, or nullptr
    int64_t *hist;        // [n][HIST_LEN] per-sweep records, or nullptr
    int32_t *tile_act;    // [1]: active bonds of the last sweep
    int32_t *tile_ncl;    // [1]: clusters of the last sweep
    uint32_t tm1, tany, k0, k1, sid, q, t0;
    int ising, n;
    uint32_t *words;      // [n][chunks][64] random words of the sweeps (small_word), or nullptr
};

// Row of site i < 2^13 in a lattice of width W <= 128: the float quotient is
// at least 0.5 / W away from the next integer, far above its rounding error.
__device__ __forceinline__ int small_row(int i, float inv_w) { return static_cast<int>((i + 0.5f) * inv_w); }

constexpr int SMALL_NT = 1024;  // 16 waves: more LDS round trips in flight on the one CU

// The random words of sites i0 (even) and i0 + 1 in sweep t, as they are used:
// bits 0 .. 3 whether the right and down bonds of the two would be active
// between equal spins, bytes 2 and 3 the states they would draw as roots.
__device__ __forceinline__ uint32_t small_word(uint32_t i0, uint32_t t, const SmallArgs &a)
{
    const U4 b = philox4x32_10(i0 >> 1, t, TAG_BOND, a.sid, a.k0, a.k1);
    const U4 f = philox4x32_10(i0 >> 2, t, TAG_FLIP, a.sid, a.k0, a.k1);
    const uint32_t on = (b.v0 <= a.tm1 ? 1u : 0u) | (b.v1 <= a.tm1 ? 2u : 0u) | (b.v2 <= a.tm1 ? 4u : 0u) |
                        (b.v3 <= a.tm1 ? 8u : 0u);
    const uint32_t w0 = (i0 & 2u) ? f.v2 : f.v0, w1 = (i0 & 2u) ? f.v3 : f.v1;
    return (a.tany ? on : 0u) | (draw_state(w0, a.q) << 16) | (draw_state(w1, a.q) << 24);
}

// LDS of a lattice swept whole by an NT_-thread workgroup (at most SITES sites).
template <int NT_, int SITES>
struct SmallSmem {
    // Per-wave list: a step adds at most 128 entries, a fuller list is worked
    // off first (workgroups of 16 waves have a CU to themselves; the others
    // share its LDS).
    static constexpr int TL = NT_ >= 1024 ? 448 : 132;
    alignas(8) int P[SITES];          // union-find parent per site, as 4 x site (read and written in pairs)
    alignas(4) uint8_t S[SITES + 4];  // states 0..q-1 (in pairs too)
    uint32_t red[NT_ / 64][12];
    uint16_t wl[NT_ / 64][TL];
};

// All a.n sweeps of a lattice of at most SITES sites (W <= SMALL_W, H <=
// SMALL_H) in one NT_-thread workgroup.
//
// The sites are taken in chunks of 128 consecutive site indices, two sites a
// lane, whatever W is: a lane's pair shares one Philox block, and rows begin
// and end anywhere in a chunk.  Right bonds inside a chunk become runs (the
// tile kernel's max-scan); every other bond is first tried as one
// compare-and-swap between the labels of its two ends, and only those that
// lose are united step by step, from per-wave lists.  The spin bytes, no longer
// needed once the bonds stand, then take the state each site would give its
// cluster; every site walks to its root and takes the root's (which the root
// itself keeps, so the bytes can be overwritten in place).  The counters of a
// record are popcounts of lane masks.
// PRE: the random words do not depend on the spins, so k_small_words has drawn
// them on the whole chip (a.words); otherwise they are drawn here.
// Bound by one workgroup's latency: chains of dependent LDS reads between three
// barriers (of 6.5 us a sweep at 64 x 64: bonds and runs 2.2, unions 2.6, walks
// and states 1.6).  Every bond united step by step, a draw at every site and
// records summed by 64-bit shuffles took 13.4 us a sweep with its record, this
// with the words drawn in the kernel 8.3, drawn ahead 6.6; 128 x 64 without
// records, 4 sweeps: 87 -> 42 us.
template <int NT_, int SITES, bool PRE>
__device__ __forceinline__ void small_body(const SmallArgs &a, SmallSmem<NT_, SITES> &sm)
{
    constexpr int NT = NT_, NWAVE = NT_ / 64;
    constexpr int MAXM = (SITES / 128 + NWAVE - 1) / NWAVE;  // chunks per wave
    constexpr int U = MAXM <= 4 ? MAXM : 1;  // chunks worked at once (more would not fit the registers)
    constexpr int TL = SmallSmem<NT_, SITES>::TL;
    static_assert(alignof(SmallSmem<NT_, SITES>) >= alignof(int2), "entries are read in pairs");
    static_assert(SITES % 128 == 0 && MAXM <= 8 && SITES <= 1 << 13, "four bits a chunk, 13-bit sites");
    int *P = sm.P;
    uint8_t *S = sm.S;
    auto &red = sm.red;
    const int W = a.W, H = a.H, N = W * H;
    const int lane = threadIdx.x & 63, wave = wave_id();
    const int nchunk = (N + 127) >> 7, M = (nchunk + NWAVE - 1) / NWAVE;
    const int c0 = wave * M;  // the wave's chunks c0 ... (those below nchunk)
    uint16_t *mylist = sm.wl[wave];
    auto down_of = [&](int i) { return i + W < N ? i + W : i + W - N; };
    for (int i = threadIdx.x; i < N; i += NT) {
        const uint32_t b = a.spins[i];
        S[i] = static_cast<uint8_t>(a.ising ? (b == 1u ? 1u : 0u) : b);
    }
    uint32_t ends = 0;  // bit 2m + j: site j of the lane's pair in chunk m ends a row
    {
        const float inv_w = 1.0f / static_cast<float>(W);
#pragma unroll
        for (int m = 0; m < MAXM; ++m) {
            const int i0 = (c0 + m) * 128 + 2 * lane;
            ends |= (i0 + 1 == (small_row(i0, inv_w) + 1) * W ? 1u : 0u) << (2 * m);
            ends |= (i0 + 2 == (small_row(i0 + 1, inv_w) + 1) * W ? 1u : 0u) << (2 * m + 1);
        }
    }
    __syncthreads();
    // counters of the calling wave's sites (wave-uniform)
    uint32_t nsat = 0, cnt[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    // Equal-neighbour masks of chunk m: right and down of the even and the odd
    // sites; with records their numbers and the states' are added up.
    struct Equal {
        uint64_t r0, r1, d0, d1;
    };
    auto equal_masks = [&](int m) {
        const int i0 = (c0 + m) * 128 + 2 * lane;
        const uint64_t V0 = lanes_lt(static_cast<uint32_t>(i0), static_cast<uint32_t>(N));
        const uint64_t V1 = lanes_lt(static_cast<uint32_t>(i0 + 1), static_cast<uint32_t>(N));
        const bool end0 = (ends >> (2 * m)) & 1u, end1 = (ends >> (2 * m + 1)) & 1u;
        const uint32_t pair = *reinterpret_cast<const uint16_t *>(&S[i0]);
        const uint32_t s0 = pair & 0xFFu, s1 = pair >> 8;
        // (lanes past the lattice read some byte of S and are masked out)
        const uint32_t x0 = (W & 1) && end0 ? S[max(i0 + 1 - W, 0)] : s1;
        const uint32_t x1 = S[end1 ? max(i0 + 2 - W, 0) : i0 + 2];
        const uint32_t y0 = S[min(down_of(i0), SITES - 1)], y1 = S[min(down_of(i0 + 1), SITES - 1)];
        Equal e;
        e.r0 = lanes_eq(s0, x0) & V0;
        e.r1 = lanes_eq(s1, x1) & V1;
        e.d0 = lanes_eq(s0, y0) & V0;
        e.d1 = lanes_eq(s1, y1) & V1;
        if (a.hist) {
            nsat += __popcll(e.r0) + __popcll(e.r1) + __popcll(e.d0) + __popcll(e.d1);
            cnt[0] += __popcll(lanes_eq(s0, 0u) & V0) + __popcll(lanes_eq(s1, 0u) & V1);
            if (a.q == 2u) {
                cnt[1] += __popcll(lanes_ne(s0, 0u) & V0) + __popcll(lanes_ne(s1, 0u) & V1);
            } else {
#pragma unroll
                for (int k = 1; k < 8; ++k) cnt[k] += __popcll(lanes_eq(s0, k) & V0) + __popcll(lanes_eq(s1, k) & V1);
            }
        }
        return e;
    };
    auto put_record = [&](uint32_t act, uint32_t ncl) {
        if (lane != 0) return;
        uint32_t *r = red[wave];
        r[0] = act;
        r[1] = ncl;
        r[2] = nsat;
#pragma unroll
        for (int k = 0; k < 8; ++k) r[3 + k] = cnt[k];
    };
    // after a barrier: thread k < 11 writes field k of the record of `sweep`
    auto write_record = [&](int sweep, bool last) {
        if (threadIdx.x >= 11) return;
        const int k = threadIdx.x;
        uint32_t tot = 0;
#pragma unroll
        for (int w = 0; w < NWAVE; ++w) tot += red[w][k];
        if (a.hist) {
            int64_t *row = a.hist + static_cast<int64_t>(sweep) * HIST_LEN;
            const int col = k == 0 ? HIST_ACTIVE : k == 1 ? HIST_NCLUST : k == 2 ? HIST_NSAT : HIST_COUNTS + k - 3;
            row[col] = static_cast<int64_t>(tot);
            if (k == 0) row[HIST_MAXCL] = -1;
        }
        if (last && k == 0) a.tile_act[0] = static_cast<int32_t>(tot);
        if (last && k == 1) a.tile_ncl[0] = static_cast<int32_t>(tot);
    };
    // Unite the n listed bonds (site | kind << 13; kind 0: down, 1: the next
    // site, 2: the row's first site), lanes refilled from the list.
    auto unite_list = [&](int n) {
        wave_lds_fence();
        int i = lane, u = 0, v = 0;
        auto next = [&]() {
            const int e = mylist[i], s = e & 0x1FFF, kind = e >> 13;
            u = lds_ld(&P[s]);
            v = lds_ld(&P[kind == 0 ? down_of(s) : kind == 1 ? s + 1 : s + 1 - W]);
        };
        if (i < n) next();
        while (i < n) {
            int done;
            unite_step(P, u, v, done);
            if (done) {
                i += 64;
                if (i < n) next();
            }
        }
        wave_lds_fence();
    };
    uint32_t prev_act = 0, prev_ncl = 0;
    uint32_t next_word[PRE ? MAXM : 1];  // of the next sweep, loaded a sweep ahead
    auto load_words = [&](int sweep) {
#pragma unroll
        for (int m = 0; m < MAXM; ++m)
            next_word[m] = a.words[(static_cast<size_t>(sweep) * nchunk + min(c0 + m, nchunk - 1)) * 64 + lane];
    };
    if constexpr (PRE) load_words(0);
    for (int sweep = 0; sweep < a.n; ++sweep) {
        const uint32_t t = a.t0 + static_cast<uint32_t>(sweep);
        const bool last = sweep + 1 == a.n;
        uint32_t act = 0, ncl = 0;
        uint32_t word[MAXM];
        uint32_t pend = 0;  // bit 4m + 2j: down bond of site j, 4m + 2j + 1: its right bond if outside the runs
#pragma unroll
        for (int k = 0; k < 8; ++k) cnt[k] = 0;
        nsat = 0;
        for (int g = 0; g < MAXM; g += U) {
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int m = g + k, c = c0 + m;
                if (m >= M || c >= nchunk) break;
                const int i0 = c * 128 + 2 * lane;
                word[m] = PRE ? next_word[m] : small_word(static_cast<uint32_t>(i0), t, a);
                const uint32_t on = word[m];
                const Equal e = equal_masks(m);
                const uint64_t mR0 = e.r0 & lanes_ne(on & 1u, 0u), mD0 = e.d0 & lanes_ne(on & 2u, 0u);
                const uint64_t mR1 = e.r1 & lanes_ne(on & 4u, 0u), mD1 = e.d1 & lanes_ne(on & 8u, 0u);
                act += __popcll(mR0) + __popcll(mR1) + __popcll(mD0) + __popcll(mD1);
                if (last && a.bonds_out) {
                    const uint32_t b0 = lane_bit(mR0, lane) | (lane_bit(mD0, lane) << 1);
                    const uint32_t b1 = lane_bit(mR1, lane) | (lane_bit(mD1, lane) << 1);
                    if (i0 < N) a.bonds_out[i0] = static_cast<uint8_t>(b0);
                    if (i0 + 1 < N) a.bonds_out[i0 + 1] = static_cast<uint8_t>(b1);
                }
                // runs: right bonds that neither end a row nor leave the chunk
                const uint64_t E0 = lanes_ne((ends >> (2 * m)) & 1u, 0u), E1 = lanes_ne((ends >> (2 * m + 1)) & 1u, 0u);
                const uint64_t out0 = mR0 & E0, out1 = mR1 & (E1 | 1ull << 63);
                const EO R = EO{mR0 & ~out0, mR1 & ~out1};
                pend |= ((lane_bit(mD0, lane) ? 1u : 0u) | (lane_bit(out0, lane) ? 2u : 0u) |
                         (lane_bit(mD1, lane) ? 4u : 0u) | (lane_bit(out1, lane) ? 8u : 0u)) << (4 * m);
                const bool e_start = lane_bit(~(R.o << 1), lane), o_start = lane_bit(~R.e, lane);
                const int x4 = 8 * lane, base4 = 512 * c;
                const int below4 = wave_max_below(o_start ? x4 + 4 : (e_start ? x4 : 0));
                const int n0 = base4 + (e_start ? x4 : below4);
                *reinterpret_cast<int2 *>(&P[i0]) = make_int2(n0, o_start ? base4 + x4 + 4 : n0);
            }
        }
        if (sweep > 0 && a.hist) put_record(prev_act, prev_ncl);  // the previous sweep's record
        __syncthreads();
        if (sweep > 0 && a.hist) write_record(sweep - 1, false);
        if constexpr (PRE)
            if (!last) load_words(sweep + 1);
        // every down bond: the higher of its ends' labels, if still a root, is
        // linked below the other (a parent stays below its child)
        int ncon = 0;
        for (int g = 0; g < MAXM; g += U) {
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int m = g + k, c = c0 + m;
                if (m >= M || c >= nchunk) break;
                const int i0 = c * 128 + 2 * lane;
                *reinterpret_cast<uint16_t *>(&S[i0]) = static_cast<uint16_t>(word[m] >> 16);
                const uint32_t bits = pend >> (4 * m);
                const int u0 = lds_ld(&P[i0]), u1 = lds_ld(&P[i0 + 1]);
                const int v0 = lds_ld(&P[min(down_of(i0), SITES - 1)]), v1 = lds_ld(&P[min(down_of(i0 + 1), SITES - 1)]);
                const int hi0 = max(u0, v0), lo0 = min(u0, v0), hi1 = max(u1, v1), lo1 = min(u1, v1);
                int got0 = hi0, got1 = hi1;
                if ((bits & 1u) && hi0 != lo0) got0 = link_root(P, hi0, lo0);
                if ((bits & 4u) && hi1 != lo1) got1 = link_root(P, hi1, lo1);
                const EO lost = EO{lanes_ne(static_cast<uint32_t>(got0), static_cast<uint32_t>(hi0)) &
                                       lanes_ne(static_cast<uint32_t>(got0), static_cast<uint32_t>(lo0)),
                                   lanes_ne(static_cast<uint32_t>(got1), static_cast<uint32_t>(hi1)) &
                                       lanes_ne(static_cast<uint32_t>(got1), static_cast<uint32_t>(lo1))};
                const EO out = EO{lanes_ne(bits & 2u, 0u), lanes_ne(bits & 8u, 0u)};
                if (ncon > TL - 128) {
                    unite_list(ncon);
                    ncon = 0;
                }
                eo_append(mylist, ncon, lost, i0, i0 + 1);
                if ((out.e | out.o) != 0ull) {
                    if (ncon > TL - 128) {
                        unite_list(ncon);
                        ncon = 0;
                    }
                    eo_append(mylist, ncon, out, i0 | 2 << 13, (i0 + 1) | ((ends >> (2 * m + 1)) & 1u ? 2 << 13 : 1 << 13));
                }
            }
        }
        unite_list(ncon);
        __syncthreads();
        // every site's root, by pointer jumping (the trees are final: every
        // entry only moves up its chain; the chains of a lane's sites are
        // walked at once; lanes past the lattice are roots of their own)
        for (int g = 0; g < MAXM; g += U) {
            int x0[U], x1[U];
#pragma unroll
            for (int m = 0; m < U; ++m) {
                const int2 x = *reinterpret_cast<const int2 *>(&P[(min(c0 + g + m, nchunk - 1)) * 128 + 2 * lane]);
                x0[m] = x.x;
                x1[m] = x.y;
            }
            for (bool more = true; more;) {
                more = false;
#pragma unroll
                for (int m = 0; m < U; ++m) {
                    const int p0 = lds_ld(lds_entry(P, x0[m])), p1 = lds_ld(lds_entry(P, x1[m]));
                    more |= (p0 != x0[m]) | (p1 != x1[m]);
                    x0[m] = p0;
                    x1[m] = p1;
                    *reinterpret_cast<int2 *>(&P[(min(c0 + g + m, nchunk - 1)) * 128 + 2 * lane]) = make_int2(p0, p1);
                }
            }
#pragma unroll
            for (int m = 0; m < U; ++m) {
                const int c = c0 + g + m;
                if (g + m >= M || c >= nchunk) break;
                const int i0 = c * 128 + 2 * lane;
                const uint32_t s0 = S[x0[m] >> 2], s1 = S[x1[m] >> 2];
                *reinterpret_cast<uint16_t *>(&S[i0]) = static_cast<uint16_t>(s0 | (s1 << 8));
                ncl += __popcll(lanes_eq(static_cast<uint32_t>(x0[m]), static_cast<uint32_t>(4 * i0)) &
                                lanes_lt(static_cast<uint32_t>(i0), static_cast<uint32_t>(N))) +
                       __popcll(lanes_eq(static_cast<uint32_t>(x1[m]), static_cast<uint32_t>(4 * i0 + 4)) &
                                lanes_lt(static_cast<uint32_t>(i0 + 1), static_cast<uint32_t>(N)));
                if (last && a.labels) {
                    if (i0 < N) a.labels[i0] = x0[m] >> 2;
                    if (i0 + 1 < N) a.labels[i0 + 1] = x1[m] >> 2;
                }
            }
        }
        __syncthreads();
        prev_act = act;
        prev_ncl = ncl;
    }
    {
        // the last sweep's record, from the final spins
        nsat = 0;
#pragma unroll
        for (int k = 0; k < 8; ++k) cnt[k] = 0;
        if (a.hist) {
#pragma unroll 1
            for (int m = 0; m < MAXM; ++m) {
                if (m >= M || c0 + m >= nchunk) break;
                (void)equal_masks(m);
            }
        }
        put_record(prev_act, prev_ncl);
        __syncthreads();
        write_record(a.n - 1, true);
    }
    for (int i = threadIdx.x; i < N; i += NT) {
        const uint32_t st = S[i];
        a.spins[i] = static_cast<uint8_t>(a.ising ? 2u * st - 1u : st);
    }
}

template <bool PRE>
__global__ __launch_bounds__(SMALL_NT) void k_small(SmallArgs a)
{
    __shared__ SmallSmem<SMALL_NT, SMALL_SITES> sm;
    small_body<SMALL_NT, SMALL_SITES, PRE>(a, sm);
}

// The words of a.n sweeps from a.t0 on: a wave per chunk and sweep.
__global__ __launch_bounds__(256) void k_small_words(SmallArgs a)
{
    const int nchunk = (a.W * a.H + 127) >> 7, lane = threadIdx.x & 63;
    const int job = static_cast<int>(blockIdx.x) * 4 + wave_id(), sweep = job / nchunk, c = job - sweep * nchunk;
    if (sweep >= a.n) return;
    a.words[static_cast<size_t>(job) * 64 + lane] =
        small_word(static_cast<uint32_t>(c * 128 + 2 * lane), a.t0 + static_cast<uint32_t>(sweep), a);
}

// --------------------------------------------------------------- digest ---

// Check-sum of an array: the sum over i of the low 64 bits of the Philox block
// at counter (i, a_i, DIGEST_TAG, 0) under the zero key, modulo 2^64.  The sum
// is order-independent, so the grid-stride partial sums may add in any order.
constexpr uint32_t DIGEST_TAG = 0xD16E57u;
enum { DIG_U8 = 0, DIG_ISING_I8 = 1, DIG_I32 = 2 };  // a_i: byte, Ising state (+1 -> 1), int32 bits

template <int KIND>
__global__ __launch_bounds__(NT) void k_digest(const void *v, int64_t n, unsigned long long *out)
{
    __shared__ unsigned long long red[NWAVE];
    unsigned long long acc = 0;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * NT + threadIdx.x; i < n;
         i += static_cast<int64_t>(gridDim.x) * NT) {
        uint32_t x;
        if constexpr (KIND == DIG_I32) {
            x = static_cast<const uint32_t *>(v)[i];
        } else {
            const uint32_t b = static_cast<const uint8_t *>(v)[i];
            x = KIND == DIG_ISING_I8 ? (b == 1u ? 1u : 0u) : b;
        }
        const U4 r = philox4x32_10(static_cast<uint32_t>(i), x, DIGEST_TAG, 0u, 0u, 0u);
        acc += static_cast<unsigned long long>(r.v0) | (static_cast<unsigned long long>(r.v1) << 32);
    }
    acc = wave_sum(acc);
    const int lane = threadIdx.x & 63, wave = wave_id();
    if (lane == 0) red[wave] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long t = 0;
        for (int w = 0; w < NWAVE; ++w) t += red[w];
        add_stat(out, t);
    }
}

// ------------------------------------------------ batched labeling requests --
//
// Many labeling requests (the served workload) in one launch per phase: each
// request keeps its input, outputs and per-tile arrays in its own memory; the
// launch's workgroups find their request through a tile -> request table, and
// index the request's arrays with the tile's index inside the request.

struct ReqDesc {
    Grid g;
    int32_t tile0;            // first tile of the request in the launch
    const uint8_t *in;
    int32_t *labels, *roots, *sizes, *n_clusters;  // roots / sizes nullptr without sizes
    int32_t *n_host;          // the count again, in host memory, or nullptr
    uint16_t *codes, *edges;
    int32_t *gkey, *gparent, *gsize, *nb, *tile_ncl;
    uint64_t *xbits;
    int32_t *row_count, *rl_slot, *rl_size;  // with sizes
};

struct ReqBatch {
    const ReqDesc *req;
    const int32_t *req_of_tile;  // launch tile -> request
    int32_t ntiles;              // tiles of all requests
};

__device__ __forceinline__ const ReqDesc &req_of(const ReqBatch &rb, int t, int &lt)
{
    const ReqDesc &R = rb.req[rb.req_of_tile[t]];
    lt = t - R.tile0;
    return R;
}

template <int MODE, int TH_, int RPW_>
__global__ __launch_bounds__(64 * TH_ / RPW_) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_tile_reqs(ReqBatch rb)
{
    static_assert(tile_fits<MODE, TH_, RPW_>, "8 waves per SIMD");
    __shared__ TileSmem<MODE, TH_, RPW_> sm;
    int lt;
    const ReqDesc &R = req_of(rb, xcd_remap(blockIdx.x, rb.ntiles), lt);
    TileArgs a{};
    a.g = R.g;
    a.in = R.in;
    a.codes = R.codes;
    a.gkey = R.gkey;
    a.gparent = R.gparent;
    a.gsize = R.gsize;
    a.edges = R.edges;
    a.xbits = R.xbits;
    a.nb = R.nb;
    // any width: the odd-width form of the row loads serves even widths too
    tile_body<MODE, false, TH_, false, false, RPW_>(a, lt, lt, sm);
}

template <int TH_>
__global__ __launch_bounds__(1024) void k_merge_reqs(ReqBatch rb)
{
    constexpr int NP = MergePasses<TH_>::N;
    const int job = blockIdx.x * static_cast<int>(blockDim.x >> 6) + wave_id(), t = job / NP;
    if (t >= rb.ntiles) return;
    int lt;
    const ReqDesc &R = req_of(rb, t, lt);
    MergeArgs m{};
    m.g = R.g;
    m.edges = R.edges;
    m.xbits = R.xbits;
    m.gkey = R.gkey;
    m.gparent = R.gparent;
    merge_tile<false, TH_, 1>(m, lt, job - t * NP);
}

template <bool SIZES, int TH_, int RPW_>
__global__ __launch_bounds__(64 * TH_ / RPW_) void k_flatten_reqs(ReqBatch rb)
{
    __shared__ FlatSmem<M_BONDS_PERIODIC, SIZES, TH_, RPW_> sm;
    int lt;
    const ReqDesc &R = req_of(rb, xcd_remap(blockIdx.x, rb.ntiles), lt);
    FlatArgs f{};
    f.g = R.g;
    f.codes = R.codes;
    f.gkey = R.gkey;
    f.gparent = R.gparent;
    f.nb = R.nb;
    f.labels = R.labels;
    f.tile_ncl = R.tile_ncl;
    f.gsize = R.gsize;
    f.row_count = R.row_count;
    f.rl_slot = R.rl_slot;
    f.rl_size = R.rl_size;
    flatten_body<M_BONDS_PERIODIC, SIZES, TH_, RPW_>(f, lt, lt, sm);
}

template <int TH_>
__global__ __launch_bounds__(NT) void k_emit_reqs(ReqBatch rb)
{
    int lt;
    const ReqDesc &R = req_of(rb, xcd_remap(blockIdx.x, rb.ntiles), lt);
    EmitArgs e{};
    e.g = R.g;
    e.row_count = R.row_count;
    e.rl_slot = R.rl_slot;
    e.rl_size = R.rl_size;
    e.gsize = R.gsize;
    e.roots = R.roots;
    e.sizes = R.sizes;
    e.max_size = nullptr;
    e.n_clusters = R.n_clusters;
    e.n_host = R.n_host;
    emit_body<TH_, true>(e, lt);
}

// Without sizes, one workgroup per request adds up its tiles' cluster counts.
__global__ __launch_bounds__(NT) void k_count_reqs(const ReqDesc *req)
{
    const ReqDesc &R = req[blockIdx.x];
    __shared__ uint32_t part[NWAVE];
    uint32_t acc = 0;
    for (int k = threadIdx.x; k < R.g.ntiles; k += NT) acc += static_cast<uint32_t>(R.tile_ncl[k]);
    acc = wave_sum_u32(acc);
    if ((threadIdx.x & 63) == 0) part[wave_id()] = acc;
    __syncthreads();
    if (threadIdx.x == 0 && R.n_clusters) {
        uint32_t t = 0;
        for (int w = 0; w < NWAVE; ++w) t += part[w];
        *R.n_clusters = static_cast<int32_t>(t);
        if (R.n_host) *R.n_host = static_cast<int32_t>(t);
    }
}

// ------------------------------------------------------ fused batch sweep ---
//
// One launch per sweep of a whole batch of independent lattices.  Workgroups
// take work items from a queue (a ticket counter) in a fixed order:
//   1. lattices small enough to be swept whole in one workgroup's LDS,
//   2. tiles of the other lattices (bond activation + tile labeling),
//   3. merge groups (up to NWAVE tiles of one lattice, a wave each),
//   4. tiles again (flatten + flip),
// with the tiled lattices in the same order in 2-4.  A merge group waits
// until every tile of its lattice is done, a flatten until every merge group
// of its lattice is done.  Items are handed out in queue order, so every item
// a workgroup waits for was taken earlier by a workgroup that is running and
// itself waits only on items taken before that: the launch needs neither a
// co-resident grid nor a grid-wide barrier, and lattices pipeline (one
// lattice's flatten runs while another's tiles are still labeled).
//
// The counters only grow: every launch takes exactly n_items + gridDim.x
// tickets (each workgroup ends on its first ticket past the items), adds
// ntiles / nmerge to a lattice's counters and gridDim.x to the exit count, so
// a launch finds its place from its first ticket and needs no reset (graph
// replays hold no memset nodes).  The last workgroup to leave advances the
// sweep counter t that the next launch reads.

constexpr unsigned long long FUSED_SPIN_LIMIT = 1ull << 24;  // dependency polls before giving up

struct FusedArgs {
    TileArgs ta;                     // tile arrays and the batch tables (ta.b)
    MergeArgs ma;
    FlatArgs fa;
    const int32_t *small_lat;        // [n_small] lattice of each whole-in-LDS item
    const int32_t *ftile;            // [n_tiles] batch tile of each tile / flatten item
    const int2 *mgroup;              // [n_mgroups] (first batch tile, number of tiles)
    unsigned long long *ticket;      // queue position
    unsigned long long *tiles_done;  // [nlat] tile items finished
    unsigned long long *merge_done;  // [nlat] merge groups finished
    unsigned long long *exit_ctr;    // workgroups finished
    uint32_t *t;                     // sweep counter (the same word as ta.b.t)
    int32_t *fault;                  // set when a dependency wait gave up (results invalid)
    int32_t n_small, n_tiles, n_mgroups;
};

// Thread 0 waits until *p >= target with an acquire at agent scope; the
// workgroup barrier then passes what it acquired on to the other waves.  On a
// chip of several XCDs an agent-scope acquire invalidates the CU's L1 and the
// XCD's L2, so it is taken once per item, by one thread.
__device__ __forceinline__ void fused_wait(const unsigned long long *p, unsigned long long target, int32_t *fault)
{
    if (threadIdx.x == 0) {
        for (unsigned long long k = 0;; ++k) {
            if (__hip_atomic_load(p, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) >= target) break;
            if (k == FUSED_SPIN_LIMIT) {
                // a bounded wait: a broken invariant ends the launch instead of hanging it
                __hip_atomic_store(fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
    }
    __syncthreads();
}

// The workgroup barrier orders every wave's writes before thread 0's
// agent-scope release, which publishes them with the count (a release writes
// the XCD's L2 back, so it too is issued once per item).
__device__ __forceinline__ void fused_signal(unsigned long long *p)
{
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_fetch_add(p, 1ull, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
}

// Lattices swept whole in LDS by a fused launch: at most this many sites (and
// W <= SMALL_W, H <= SMALL_H), so their LDS (5 bytes a site) fits the tile
// phase's budget per workgroup.
template <int NT_>
struct FusedSmall {
    static constexpr int SITES = NT_ * 15 < 7680 ? NT_ * 15 : 7680;
};

template <int TH_>
__global__ __launch_bounds__(Tile<TH_>::NT) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_batch_fused(FusedArgs a)
{
    using S = Tile<TH_>;
    constexpr int NT = S::NT, NWAVE = S::NWAVE, SMALL = FusedSmall<NT>::SITES;
    __shared__ union {
        TileSmem<M_SW, TH_> tile;
        FlatSmem<M_SW, false, TH_> flat;
        SmallSmem<NT, SMALL> small;
    } sm;
    __shared__ unsigned long long ticket_s;
    static_assert(sizeof(sm) + sizeof(ticket_s) <= LDS_PER_WAVE * NWAVE, "8 waves per SIMD");
    const uint32_t t = *a.t;  // every workgroup reads it before the last one leaves and advances it
    const long long n_items = static_cast<long long>(a.n_small) + 2ll * a.n_tiles + a.n_mgroups;
    const unsigned long long per_launch = static_cast<unsigned long long>(n_items) + gridDim.x;
    unsigned long long base = 0, launch = 0;
    for (bool first = true;; first = false) {
        if (threadIdx.x == 0) ticket_s = __hip_atomic_fetch_add(a.ticket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        const unsigned long long tk = uniform64(ticket_s);  // wave-uniform: the item's loads are scalar
        __syncthreads();
        if (first) {
            launch = tk / per_launch;
            base = launch * per_launch;
        }
        long long item = static_cast<long long>(tk - base);
        if (item >= n_items) break;
        if (item < a.n_small) {
            const int j = __builtin_amdgcn_readfirstlane(a.small_lat[item]);
            const LatticeDesc &L = a.ta.b.lat[j];
            SmallArgs s{};
            s.W = L.g.W;
            s.H = L.g.H;
            s.spins = L.spins;
            s.bonds_out = L.bonds;
            s.labels = L.labels;
            s.hist = nullptr;
            s.tile_act = a.ta.tile_act + L.tile0;
            s.tile_ncl = a.fa.tile_ncl + L.tile0;
            s.tm1 = L.tm1;
            s.tany = L.tany;
            s.k0 = L.k0;
            s.k1 = L.k1;
            s.sid = L.sid;
            s.q = L.q;
            s.t0 = t;
            s.ising = L.ising;
            s.n = 1;
            small_body<NT, SMALL, false>(s, sm.small);
            __syncthreads();  // the LDS is reused by the next item
            continue;
        }
        item -= a.n_small;
        if (item < a.n_tiles) {
            const int tile = __builtin_amdgcn_readfirstlane(a.ftile[item]);
            TileArgs ta = a.ta;
            int lt;
            load_batch_tile(ta, tile, lt);
            if (ta.g.W % 2 == 0)
                tile_body<M_SW, true, TH_>(ta, tile, lt, sm.tile);
            else
                tile_body<M_SW, false, TH_>(ta, tile, lt, sm.tile);
            fused_signal(&a.tiles_done[a.ta.b.lat_of_tile[tile]]);
            continue;
        }
        item -= a.n_tiles;
        if (item < a.n_mgroups) {
            const int2 g2 = a.mgroup[item];
            const int2 grp = make_int2(__builtin_amdgcn_readfirstlane(g2.x), __builtin_amdgcn_readfirstlane(g2.y));
            const int j = a.ta.b.lat_of_tile[grp.x];
            const LatticeDesc &L = a.ta.b.lat[j];
            fused_wait(&a.tiles_done[j], (launch + 1) * static_cast<unsigned long long>(L.g.ntiles), a.fault);
            const int w = wave_id();
            if (w < grp.y) merge_tile<true, TH_, MergePasses<TH_>::N>(a.ma, grp.x + w, 0);
            fused_signal(&a.merge_done[j]);
            continue;
        }
        item -= a.n_mgroups;
        {
            const int tile = __builtin_amdgcn_readfirstlane(a.ftile[item]);
            const int j = a.ta.b.lat_of_tile[tile];
            fused_wait(&a.merge_done[j], (launch + 1) * static_cast<unsigned long long>(a.ta.b.lat[j].nmerge),
                       a.fault);
            FlatArgs fa = a.fa;
            int lt;
            load_batch_flat(fa, tile, lt);
            flatten_body<M_SW, false, TH_>(fa, tile, lt, sm.flat);
            __syncthreads();  // the LDS is reused by the next item
        }
    }
    if (threadIdx.x == 0) {
        __threadfence();
        const unsigned long long left = __hip_atomic_fetch_add(a.exit_ctr, 1ull, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) + 1;
        if (left % gridDim.x == 0) __hip_atomic_store(a.t, t + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

}  // namespace swccl

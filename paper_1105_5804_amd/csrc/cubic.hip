// cubic.hip -- the SW sweep on the periodic simple cubic lattice: the same
// three steps as on the square lattice (Sec. II), generalised to three
// dimensions, and the host side of the sw3_* calls of include/swccl.h.
//
// A sweep is four launches:
//
//   k3_tile     one 512-thread workgroup per 32 x 16 x 16 tile (the shape of
//               8192 sites with the fewest face sites and crossing bonds);
//               two sites per lane, a wave-wide step covering one row of four
//               z-planes, each wave eight steps along y.
//               Bond activation of the +x, +y and +z bonds (Sec. II.A) fused
//               with the tile's labeling (Sec. II.B.2): labels handed along
//               x runs, down the rows and across planes, the bonds left over
//               united by a lock-free union-find in LDS; the clusters touching
//               any tile face are claimed and get compact ids; every site gets
//               a 16-bit code (the slot of its interior root, or CSITES + its
//               cluster's id; the crossing bonds in the bits above).
//   k3_merge    every active bond that leaves a tile through its +x, +y or +z
//               face (periodic wraps included) unites two ids in the global
//               union-find (Sec. II.C).  Roots are linked by a fixed random
//               priority of the ids rather than by key: on the cubic lattice
//               at criticality key-ordered links build trees too deep to walk
//               for the ~10^7 ids of a sweep.
//   k3_resolve  every id pointed at its root, and the cluster's minimum site
//               index (its canonical label) gathered at the root's key;
//   k3_flatten  one draw per cluster at that index (Sec. II.D): the tile's ids
//               and its interior roots, then every site's new state (and
//               optionally label) from its code.
//
// With per-sweep records, k_observe counts the satisfied bonds and states of
// the new spins, adds up the tiles' counters and writes the record.
//
// ccl3_label runs the same tile, merge, resolve and flatten kernels on given
// bond bytes (LABEL = true): no spins, no draws, labels out.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "../../include/swccl.h"
#include "internal.hpp"
#include "observe.hpp"
#include "philox.hpp"
#include "uf.hpp"

namespace swccl {
namespace cubic {

constexpr int CX = 32, CY = 16, CZ = 16;                      // tile extent (x fastest)
constexpr int PLANE = CX * CY;                                 // sites of a tile z-plane
constexpr int CSITES = PLANE * CZ;                             // sites per tile
constexpr int CAP = CSITES - (CX - 2) * (CY - 2) * (CZ - 2);   // sites on a face of a full tile
// Lanes: two sites each, so a wave-wide step covers 128 sites: one row of
// each of SUB z-planes.  NW3 waves: wave w takes the planes (w / 2) SUB ... of
// y range (w mod 2) ITER ..., ITER steps down its rows.
constexpr int NW3 = 8;                                         // waves per tile workgroup
constexpr int NT3 = 64 * NW3;
constexpr int LPR = CX / 2;                                    // lanes per tile row
constexpr int SUB = 64 / LPR;                                  // tile rows (planes) per step
constexpr int RPI = SUB;
constexpr int ITER = 8;                                        // steps per wave
constexpr int TL3 = 448;                                       // per-wave lists: a step adds at most 128 entries at a
                                                               // time, a fuller list is worked off first
static_assert(CSITES == 128 * NW3 * ITER && CY == 2 * ITER && CZ == SUB * NW3 / 2, "the waves cover the tile");
constexpr int MSEEN = 1024;                                    // merge: pair-dedup slots per face
constexpr int FX = CY * CZ, FY = CX * CZ, FZ = CX * CY;        // sites of the +x, +y, +z faces
constexpr uint32_t TAG_BOND = 1, TAG_FLIP = 2, TAG_BOND_Z = 5;
// A code is the slot of the site's interior root or CSITES + its id; the two
// bits above carry the +y and +z bonds of sites on the last row and plane.
constexpr uint32_t CODE_MASK = 0x3FFF;
static_assert(CAP + CSITES <= CODE_MASK, "codes take 14 bits");
static_assert(CAP < (1 << 15), "merge list entries hold two ids in 15 bits each");

struct Geo3 {
    int Lx, Ly, Lz;
    int ntx, nty, ntz, ntiles;
};

// Tile of a workgroup and its extent (ragged at the +x, +y, +z ends).
struct TileOf {
    int tile, gx0, gy0, gz0, tw, th, td;
};
__device__ __forceinline__ TileOf tile_of(const Geo3 &g, int tile)
{
    const int tx = tile % g.ntx, ty = (tile / g.ntx) % g.nty, tz = tile / (g.ntx * g.nty);
    TileOf t;
    t.tile = tile;
    t.gx0 = tx * CX;
    t.gy0 = ty * CY;
    t.gz0 = tz * CZ;
    t.tw = min(CX, g.Lx - t.gx0);
    t.th = min(CY, g.Ly - t.gy0);
    t.td = min(CZ, g.Lz - t.gz0);
    return t;
}

// Position of site (lx, ly, lz) in a tile's code array: the order in which the
// waves' steps write and read them, 256 contiguous bytes a step.
__device__ __forceinline__ int code_pos(int lx, int ly, int lz)
{
    const int w = lz / SUB * 2 + ly / ITER;
    return ((w * ITER + ly % ITER) * 64 + lz % SUB * LPR) * 2 + lx;
}

// Site index of tile slot s = (lz CY + ly) CX + lx.
__device__ __forceinline__ int32_t site_of(const Geo3 &g, const TileOf &t, int s)
{
    const int lz = s / PLANE, ly = (s / CX) % CY, lx = s % CX;
    return static_cast<int32_t>((static_cast<int64_t>(t.gz0 + lz) * g.Ly + t.gy0 + ly) * g.Lx + t.gx0 + lx);
}

// Value of x held by the other lane of the calling lane's pair (2m <-> 2m + 1;
// DPP quad permutation 1, 0, 3, 2).
__device__ __forceinline__ uint32_t swap_pair_lanes(uint32_t x)
{
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0xB1, 0xF, 0xF, false));
}

// Maximum of v >= 0 over the lanes below the calling one in its group of 16
// (0 for the first): a max-scan by row shifts (a DPP row is 16 lanes, LPR of
// them a tile row), then a shift by one lane.
static_assert(LPR == 16, "a tile row is a DPP row");
__device__ __forceinline__ int row_max_below(int v)
{
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false));  // row_shr:1
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false));  // row_shr:2
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false));  // row_shr:4
    v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false));  // row_shr:8
    return __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);
}

struct Tile3Args {
    Geo3 g;
    const uint8_t *in;        // spins, or the given bonds (LABEL)
    uint8_t *bonds;           // [N] packed bonds of the sweep (bit0 +x, bit1 +y, bit2 +z), or nullptr
    uint16_t *codes;          // [ntiles][CSITES], in the order of code_pos
    uint16_t *xface;          // [ntiles][2][FX]: ids of the x = 0 sites, then of the x = tw - 1 sites | +x bond << 15
    int32_t *gkey, *gparent;  // [ntiles][CAP]
    int32_t *nb;              // [ntiles]: ids of the tile
    int32_t *tile_act;        // [ntiles]: active bonds owned by the tile
    uint32_t tm1, tany;       // a bond is active iff its word r <= tm1 and tany (T > 0; tm1 = T - 1)
    uint32_t k0, k1, t, sid;
    uint32_t *ticket;         // cleared for the observables that follow, or nullptr
};

// Slot of face position t (the z, then y, then x faces of a full tile), or -1
// outside a ragged tile.
constexpr int FACES = 2 * (FZ + FY + FX);
__device__ __forceinline__ int face_slot(int t, const TileOf &T)
{
    int lx, ly, lz;
    if (t < 2 * FZ) {
        lx = t % CX;
        ly = t / CX % CY;
        lz = t < FZ ? 0 : T.td - 1;
    } else if (t < 2 * (FZ + FY)) {
        t -= 2 * FZ;
        lx = t % CX;
        lz = t / CX % CZ;
        ly = t < FY ? 0 : T.th - 1;
    } else {
        t -= 2 * (FZ + FY);
        ly = t % CY;
        lz = t / CY % CZ;
        lx = t < FX ? 0 : T.tw - 1;
    }
    return lx < T.tw && ly < T.th && lz < T.td ? lz * PLANE + ly * CX + lx : -1;
}

// LABEL: the bonds are given (a.in, only read); otherwise they are drawn from
// the spins (and written if asked for).
//
// A wave owns SUB z-planes of half a tile's y range and goes down their rows
// together: lane group `sub` holds plane sub's row, two sites a lane.  +x
// bonds become runs of a row (a max-scan over its 16 lanes), a run takes the
// label of one run before it along y by a plain LDS write, and a label still
// a root is linked below the plane before it by one compare-and-swap, as are
// the contacts with other waves' rows and planes after a barrier.  Only the
// bonds that lose (two labels already, or a root linked elsewhere) are united
// step by step.  At the critical point 0.24 of the bonds of each direction
// are active and about a tenth of them are left to unite, where uniting every
// bond inside the tile cost two thirds of the kernel.  The crossing bonds go
// out in the codes' upper bits, so no bond array is written unless asked for.
// Still bound by VALU issue: 474 -> 293 VALU instructions per 128 sites, the
// kernel 868 -> 473 us at 512^3 and beta_c, the sweep 1.539 -> 1.083 ms.
// FOUR: Lx is a multiple of 4 (pairs of sites load and store as one, and
// share random blocks); the general form serves every Lx.
// ROWS: steps (tile rows along y) of a wave; half of ITER with twice the waves
// on lattices of few tiles (see the launch).
template <bool LABEL, bool FOUR, int ROWS>
__global__ __launch_bounds__(NT3 * ITER / ROWS) __attribute__((amdgpu_waves_per_eu(8, 8))) void k3_tile(Tile3Args a)
{
    constexpr int ITER = ROWS, YW = CY / ROWS, NW3 = YW * CZ / SUB, NT3 = 64 * NW3;  // waves along y, and in all
    // union-find parent per slot, as 4 x slot (read and written in pairs)
    __shared__ alignas(8) int P[CSITES];
    __shared__ uint16_t wl[NW3][TL3];     // per-wave list: 4 x slot | direction (0 +y, 1 +z) of a bond, or a label
    __shared__ uint32_t zb[NW3][LPR];     // +z bonds of the wave's last plane: bit 2 it + j of a lane's sites
    __shared__ int nb_s;
    __shared__ unsigned act_w[NW3];
    static_assert(sizeof(P) + sizeof(wl) + sizeof(zb) + sizeof(act_w) + sizeof(nb_s) <= 160 * 1024 / 32 * NW3,
                  "8 waves per SIMD");
    const Geo3 g = a.g;
    const TileOf T = tile_of(g, xcd_remap(blockIdx.x, g.ntiles));
    const int lane = threadIdx.x & 63, w = wave_id();
    const int sub = lane / LPR, lx0 = 2 * (lane % LPR), x4 = 4 * lx0;
    const int lz = w / YW * SUB + sub, ly0 = w % YW * ITER;
    const int nr = max(0, min(ITER, T.th - ly0));  // tile rows along y owned by this wave
    const bool zin = lz < T.td;
    const bool v0 = zin && lx0 < T.tw, v1 = zin && lx0 + 1 < T.tw;
    const bool ragged = T.tw < CX || T.td < CZ;
    uint16_t *mylist = wl[w];
    if (threadIdx.x == 0) nb_s = 0;
    if (T.tile == 0 && threadIdx.x == 0 && a.ticket) *a.ticket = 0u;
    // lane masks (each tile row's 16 lanes alike): the last column's sites
    const uint32_t row0m = 0xFFFFu >> (LPR - ((T.tw + 1) >> 1)), row1m = row0m >> (T.tw & 1);
    const uint64_t every = 0x0001000100010001ull;
    const uint64_t L0 = (row0m & ~row1m) * every, L1 = (row1m & ~(row0m >> 1)) * every;

    auto unite_list = [&](int n) {  // as in the square-lattice tile
        wave_lds_fence();
        int i = lane, u = 0, v = 0;
        auto next = [&]() {
            const int e = mylist[i], c = e & ~3;
            u = lds_ld(lds_entry(P, c));
            v = lds_ld(lds_entry(P, c + ((e & 1) ? 4 * PLANE : 4 * CX)));
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
    int ncon = 0;
    auto append = [&](EO m, int e) {  // the bonds m of the sites at byte offset e (| direction)
        if (ncon > TL3 - 128) {
            unite_list(ncon);
            ncon = 0;
        }
        eo_append(mylist, ncon, m, e, e + 4);
    };

    // ---- loads of the wave's rows (site indices fit 32 bits): cur[it] is the
    // pair of bytes at tile row ly0 + it of the lane's plane (one more row for
    // the +y neighbours), zz[it] the pair in the next plane, hl[it] the byte
    // right of the tile.  Lanes outside the tile read a valid address.
    const uint32_t Lx = static_cast<uint32_t>(g.Lx), Ly = static_cast<uint32_t>(g.Ly), Lz = static_cast<uint32_t>(g.Lz);
    const uint32_t gz = static_cast<uint32_t>(T.gz0 + min(lz, T.td - 1)), gy = static_cast<uint32_t>(T.gy0 + ly0);
    const uint32_t row0 = (gz * Ly + gy) * Lx;
    const uint32_t dz = (gz + 1u == Lz ? 0u - gz : 1u) * (Ly * Lx);  // to the next plane (modulo 2^32)
    const uint32_t xs0 = static_cast<uint32_t>(T.gx0 + (lx0 < T.tw ? lx0 : 0));
    const uint32_t xs1 = static_cast<uint32_t>(T.gx0 + (lx0 + 1 < T.tw ? lx0 + 1 : 0));
    const uint32_t hx = static_cast<uint32_t>(T.gx0 + T.tw) == Lx ? 0u : static_cast<uint32_t>(T.gx0 + T.tw);
    const bool even_lx = FOUR || (Lx & 1u) == 0u;
    auto pair_at = [&](uint32_t row) -> uint32_t {
        if (even_lx) return *reinterpret_cast<const uint16_t *>(a.in + row + xs0);  // every row starts even
        return static_cast<uint32_t>(a.in[row + xs0]) | (static_cast<uint32_t>(a.in[row + xs1]) << 8);
    };
    uint32_t cur[ITER + 1], zz[ITER], hl[ITER];
#pragma unroll
    for (int it = 0; it <= ITER; ++it) {
        cur[it] = 0;
        if (it < ITER) zz[it] = hl[it] = 0;
        if (nr > 0 && (it < nr || (!LABEL && it == nr))) {
            const bool wrap = gy + static_cast<uint32_t>(it) == Ly;
            const uint32_t row = row0 + static_cast<uint32_t>(it) * Lx - (wrap ? Ly * Lx : 0u);
            cur[it] = pair_at(row);
            if (!LABEL && it < nr) {
                zz[it] = pair_at(row + dz);
                hl[it] = a.in[row + hx];
            }
        }
    }
    if (ragged) {
        // sites outside the tile have no bonds: spins that differ from each
        // other, from every byte and from the next row's (bits 8 up exceed a
        // byte in the upper site); bond bytes 0
#pragma unroll
        for (int it = 0; it <= ITER; ++it) {
            const uint32_t no0 = LABEL ? 0u : (it & 1), no1 = LABEL ? 0u : (0x102u + (it & 1)) << 8;
            cur[it] = v1 ? cur[it] : (v0 ? cur[it] & 0xFFu : no0) | no1;
            if (!LABEL && it < ITER && !v0) zz[it] = hl[it] = 0x80u;
        }
    }

    // ---- bonds and labels, row by row
    // with Lx a multiple of 4 every row starts at a multiple of 4, so the two
    // lanes of a pair share one +z block per row: each draws the block of one
    // of two consecutive rows and the halves are swapped between the pair
    constexpr bool zpairs = FOUR;
    const bool odd_lane = (lane & 1) != 0;
    uint32_t zpend0 = 0, zpend1 = 0;  // +z words of the next row, drawn with this one
    int lab0[ITER], lab1[ITER];       // labels of the lane's sites (byte offsets)
    uint32_t xbit = 0, zbit = 0;      // the lane's +x bonds that leave the tile (bit it), its +z bonds (bit 2 it + j)
    unsigned act = 0;
    EO prevY = EO{0ull, 0ull};
    const int own_first = 4 * (lz * PLANE + ly0 * CX) + x4;  // the lane's first site, as a byte offset
    const int next_plane4 = 4 * (lz + 1) * PLANE;
    const uint64_t inner = __ballot(sub < SUB - 1 && lz + 1 < T.td);  // lanes whose next plane is this wave's
#pragma unroll
    for (int it = 0; it < ITER; ++it) lab0[it] = lab1[it] = 0;
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        if (it >= nr) break;
        const uint32_t i0 = row0 + static_cast<uint32_t>(it) * Lx + static_cast<uint32_t>(T.gx0 + lx0);
        uint64_t mX0, mX1, mY0, mY1, mZ0, mZ1;
        if constexpr (LABEL) {
            const uint32_t c = cur[it];
            mX0 = lanes_ne(c & 0x001u, 0u);
            mY0 = lanes_ne(c & 0x002u, 0u);
            mZ0 = lanes_ne(c & 0x004u, 0u);
            mX1 = lanes_ne(c & 0x100u, 0u);
            mY1 = lanes_ne(c & 0x200u, 0u);
            mZ1 = lanes_ne(c & 0x400u, 0u);
        } else {
            const uint32_t s0 = cur[it] & 0xFFu, s1 = cur[it] >> 8;
            const uint32_t y0 = cur[it + 1] & 0xFFu, y1 = cur[it + 1] >> 8;
            const uint32_t z0 = zz[it] & 0xFFu, z1 = zz[it] >> 8;
            const uint32_t nxt = from_next_lane(s0);
            const uint32_t x0 = lane_bit(L0, lane) ? hl[it] : s1;
            const uint32_t x1 = lane_bit(L1, lane) ? hl[it] : nxt;
            // words: +x and +y from block(i >> 1, BOND) as on the square
            // lattice, +z word i & 3 of block(i >> 2, BOND_Z)
            uint32_t k0 = a.k0, k1 = a.k1;  // the key schedule is recomputed per row, not held across rows
            asm volatile("" : "+s"(k0), "+s"(k1));
            const U4 bk = philox4x32_10(i0 >> 1, a.t, TAG_BOND, a.sid, k0, k1);
            uint32_t rx0 = bk.v0, ry0 = bk.v1, rx1 = bk.v2, ry1 = bk.v3;
            if (!even_lx && (i0 & 1u) != 0u) {  // odd row start: i0 is the second site of its block
                rx0 = bk.v2;
                ry0 = bk.v3;
                const U4 b2 = philox4x32_10((i0 >> 1) + 1u, a.t, TAG_BOND, a.sid, k0, k1);
                rx1 = b2.v0;
                ry1 = b2.v1;
            }
            uint32_t rz0, rz1;
            if (zpairs && (it & 1) == 0) {
                // the even lane draws its pair's block of this row, the odd
                // lane that of the next row
                const uint32_t pair = i0 - (odd_lane ? 2u : 0u) + (odd_lane ? Lx : 0u);
                const U4 bz = philox4x32_10(pair >> 2, a.t, TAG_BOND_Z, a.sid, k0, k1);
                const uint32_t ra = swap_pair_lanes(odd_lane ? bz.v0 : bz.v2);
                const uint32_t rb = swap_pair_lanes(odd_lane ? bz.v1 : bz.v3);
                rz0 = odd_lane ? ra : bz.v0;  // this row: words 0, 1 (even lane) or 2, 3 (odd lane)
                rz1 = odd_lane ? rb : bz.v1;
                zpend0 = odd_lane ? bz.v2 : ra;  // the next row
                zpend1 = odd_lane ? bz.v3 : rb;
            } else if (zpairs) {
                rz0 = zpend0;
                rz1 = zpend1;
            } else {
                const U4 bz = philox4x32_10(i0 >> 2, a.t, TAG_BOND_Z, a.sid, k0, k1);
                rz0 = pick(bz, i0 & 3u);
                rz1 = pick(bz, (i0 + 1u) & 3u);
                if (((i0 + 1u) & 3u) == 0u)  // site i0 + 1 starts the next block
                    rz1 = philox4x32_10((i0 + 1u) >> 2, a.t, TAG_BOND_Z, a.sid, k0, k1).v0;
            }
            mX0 = lanes_eq(s0, x0) & lanes_le(rx0, a.tm1);
            mY0 = lanes_eq(s0, y0) & lanes_le(ry0, a.tm1);
            mZ0 = lanes_eq(s0, z0) & lanes_le(rz0, a.tm1);
            mX1 = lanes_eq(s1, x1) & lanes_le(rx1, a.tm1);
            mY1 = lanes_eq(s1, y1) & lanes_le(ry1, a.tm1);
            mZ1 = lanes_eq(s1, z1) & lanes_le(rz1, a.tm1);
            if (!a.tany) mX0 = mX1 = mY0 = mY1 = mZ0 = mZ1 = 0ull;
            act += __popcll(mX0) + __popcll(mX1) + __popcll(mY0) + __popcll(mY1) + __popcll(mZ0) + __popcll(mZ1);
            if (a.bonds) {
                const uint32_t b0 = lane_bit(mX0, lane) | (lane_bit(mY0, lane) << 1) | (lane_bit(mZ0, lane) << 2);
                const uint32_t b1 = lane_bit(mX1, lane) | (lane_bit(mY1, lane) << 1) | (lane_bit(mZ1, lane) << 2);
                if (even_lx && v1) {
                    *reinterpret_cast<uint16_t *>(a.bonds + i0) = static_cast<uint16_t>(b0 | (b1 << 8));
                } else {
                    if (v0) a.bonds[i0] = static_cast<uint8_t>(b0);
                    if (v1) a.bonds[i0 + 1] = static_cast<uint8_t>(b1);
                }
            }
        }
        // bonds that leave the tile: +x of the last column, +y of the last row
        // (the next wave's rows excepted, after the loop), +z of the last plane
        xbit |= lane_bit((mX0 & L0) | (mX1 & L1), lane) ? 1u << it : 0u;
        zbit |= (lane_bit(mZ0, lane) ? 1u << (2 * it) : 0u) | (lane_bit(mZ1, lane) ? 2u << (2 * it) : 0u);
        const EO R = EO{mX0 & ~L0, mX1 & ~L1};
        // run starts in the row, as byte offsets (the row's first site always
        // starts a run, at offset 0)
        const bool e_start = lane_bit(~(R.o << 1), lane);
        const bool o_start = lane_bit(~R.e, lane);
        const int below4 = row_max_below(o_start ? x4 + 4 : (e_start ? x4 : 0));
        const int own = own_first + it * 4 * CX, row4 = own - x4;
        int n0 = row4 + (e_start ? x4 : below4);
        int n1 = o_start ? own + 4 : n0;
        *reinterpret_cast<int2 *>(lds_entry(P, own)) = make_int2(n0, n1);
        if (it > 0) {
            // every +y bond offers its site's label to the next row's run
            // (one wave's LDS operations run in order; whichever offer lands
            // last stands); a bond whose label lost needs a union
            const int up0 = lab0[it > 0 ? it - 1 : 0], up1 = lab1[it > 0 ? it - 1 : 0];
            wave_lds_fence();
            if (lane_bit(prevY.e, lane)) lds_st(lds_entry(P, n0), up0);
            if (lane_bit(prevY.o, lane)) lds_st(lds_entry(P, n1), up1);
            wave_lds_fence();
            n0 = lds_ld(lds_entry(P, n0));
            n1 = lds_ld(lds_entry(P, n1));
            *reinterpret_cast<int2 *>(lds_entry(P, own)) = make_int2(n0, n1);
            append(EO{lanes_ne(static_cast<uint32_t>(n0), static_cast<uint32_t>(up0)) & prevY.e,
                      lanes_ne(static_cast<uint32_t>(n1), static_cast<uint32_t>(up1)) & prevY.o},
                   own - 4 * CX);
        }
        lab0[it] = n0;
        lab1[it] = n1;
        prevY = EO{mY0, mY1};
        {
            // +z bonds to the wave's next plane (the lanes of the next group):
            // a label there that is still a root is linked below this one
            const EO Z = EO{mZ0 & inner, mZ1 & inner};
            wave_lds_fence();
            int got0 = -1, got1 = -1, up0 = 0, up1 = 0;
            if (sub < SUB - 1) {
                up0 = lds_ld(lds_entry(P, own + 4 * PLANE));
                up1 = lds_ld(lds_entry(P, own + 4 * PLANE + 4));
            }
            if (lane_bit(Z.e, lane) && up0 >= next_plane4) got0 = link_root(P, up0, n0);
            if (lane_bit(Z.o, lane) && up1 >= next_plane4) got1 = link_root(P, up1, n1);
            const EO met = EO{lanes_eq(static_cast<uint32_t>(got0), static_cast<uint32_t>(up0)) |
                                  lanes_eq(static_cast<uint32_t>(got0), static_cast<uint32_t>(n0)),
                              lanes_eq(static_cast<uint32_t>(got1), static_cast<uint32_t>(up1)) |
                                  lanes_eq(static_cast<uint32_t>(got1), static_cast<uint32_t>(n1))};
            append(eo_andnot(Z, met), own | 1);
        }
    }
    if (sub == SUB - 1) zb[w][lane % LPR] = zin && lz + 1 < T.td ? zbit : 0u;
    __syncthreads();

    // ---- bonds to other waves' rows and planes, then all unions
    auto link_across = [&](EO m, int own, int up4, int n0, int n1, int dir) {
        // the sites at `own` with labels n0, n1 and bonds m to the sites
        // `up4` bytes on; labels there below their first slot are left to the list
        const int q0 = lds_ld(lds_entry(P, own + up4)), q1 = lds_ld(lds_entry(P, own + up4 + 4));
        const int first = dir == 0 ? own + up4 - x4 : (own + up4) & ~(4 * PLANE - 1);
        int got0 = -1, got1 = -1;
        if (lane_bit(m.e, lane) && q0 >= first) got0 = link_root(P, q0, n0);
        if (lane_bit(m.o, lane) && q1 >= first) got1 = link_root(P, q1, n1);
        const EO met = EO{lanes_eq(static_cast<uint32_t>(got0), static_cast<uint32_t>(q0)) |
                              lanes_eq(static_cast<uint32_t>(got0), static_cast<uint32_t>(n0)),
                          lanes_eq(static_cast<uint32_t>(got1), static_cast<uint32_t>(q1)) |
                              lanes_eq(static_cast<uint32_t>(got1), static_cast<uint32_t>(n1))};
        append(eo_andnot(m, met), own | dir);
    };
    if (nr == ITER && ly0 + ITER < T.th)  // the next part of the y range
        link_across(prevY, own_first + (ITER - 1) * 4 * CX, 4 * CX, lab0[ITER - 1], lab1[ITER - 1], 0);
    {
        // the wave's last plane to the next wave's first: RPI rows a step
        const int lz_last = w / YW * SUB + SUB - 1;
#pragma unroll
        for (int s = 0; s < ITER / RPI; ++s) {
            const int it = s * RPI + sub;
            const uint32_t z = zb[w][lane % LPR] >> (2 * it);
            const EO m = EO{lanes_ne(z & 1u, 0u), lanes_ne(z & 2u, 0u)};
            if ((m.e | m.o) == 0ull) continue;
            const int own = 4 * (lz_last * PLANE + (ly0 + it) * CX) + x4;
            const int n0 = lds_ld(lds_entry(P, own)), n1 = lds_ld(lds_entry(P, own + 4));
            link_across(m, own, 4 * PLANE, n0, n1, 1);
        }
    }
    unite_list(ncon);
    __syncthreads();

    // ---- claims: the root of every cluster that touches a tile face gets an id
    for (int t = threadIdx.x; t < FACES; t += NT3) {
        const int slot = face_slot(t, T);
        if (slot < 0) continue;
        const int r4 = lroot(P, 4 * slot);
        int expect = r4;
        if (__hip_atomic_compare_exchange_strong(lds_entry(P, r4), &expect, CLAIMING, __ATOMIC_RELAXED,
                                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) {
            const int k = atomicAdd(&nb_s, 1);
            lds_st(lds_entry(P, r4), final_entry(static_cast<uint32_t>(CSITES + k)));
            const int id = T.tile * CAP + k;
            a.gkey[id] = site_of(g, T, r4 >> 2);
            a.gparent[id] = id;
        }
    }
    __syncthreads();

    // ---- every linked label gets its cluster's final entry (as in the
    // square-lattice tile: a walk ends at a claimed root, at a label another
    // lane has finished, or at an unclaimed root, its own parent)
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
    int nls = 0;
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        if (it >= nr) break;
        if (nls > TL3 - 128) {
            compress_list(nls);
            nls = 0;
        }
        // a label site whose entry is an offset below its own (a final entry
        // is negative, above every offset as an unsigned number)
        const uint32_t own = static_cast<uint32_t>(own_first + it * 4 * CX);
        const int2 p = *reinterpret_cast<const int2 *>(lds_entry(P, static_cast<int>(own)));
        const EO linked = EO{lanes_eq(static_cast<uint32_t>(lab0[it]), own) & lanes_lt(static_cast<uint32_t>(p.x), own),
                             lanes_eq(static_cast<uint32_t>(lab1[it]), own + 4) &
                                 lanes_lt(static_cast<uint32_t>(p.y), own + 4)};
        eo_append(mylist, nls, linked, static_cast<int>(own), static_cast<int>(own + 4));
    }
    compress_list(nls);
    __syncthreads();

    // ---- codes: the entry of the site's label; on the tile's last row the +y
    // bond in bit 15, on its last plane the +z bond in bit 14 (all such sites
    // carry ids)
    {
        uint32_t *codes32 = reinterpret_cast<uint32_t *>(a.codes + static_cast<int64_t>(T.tile) * CSITES) +
                            (w / YW * CY + ly0) * 64 + lane;
        uint16_t *xf = a.xface + static_cast<int64_t>(T.tile) * (2 * FX) + lz * CY + ly0;
        const bool z_last = lz == T.td - 1;
#pragma unroll
        for (int it = 0; it < ITER; ++it) {
            if (it >= nr) break;
            const uint32_t c0 = entry_code(lds_ld(lds_entry(P, lab0[it])));
            const uint32_t c1 = entry_code(lds_ld(lds_entry(P, lab1[it])));
            uint32_t c = c0 | (c1 << 16);
            if (ly0 + it == T.th - 1)
                c |= (lane_bit(prevY.e, lane) ? 0x8000u : 0u) | (lane_bit(prevY.o, lane) ? 0x80000000u : 0u);
            if (z_last) c |= ((zbit >> (2 * it)) & 1u) << 14 | ((zbit >> (2 * it + 1)) & 1u) << 30;
            codes32[it * 64] = c;
            // the x faces' ids again, packed by row (the merge reads them
            // whole); a row's x-face position is lz CY + ly
            if (zin) {
                const int jl = T.tw - 1 - lx0;
                if (lx0 == 0) xf[it] = static_cast<uint16_t>(c0 - CSITES);
                if (jl == 0 || jl == 1)
                    xf[FX + it] = static_cast<uint16_t>(((jl == 0 ? c0 : c1) - CSITES) | (((xbit >> it) & 1u) << 15));
            }
        }
    }
    if (lane == 0) act_w[w] = act;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned sum = 0;
        for (int k = 0; k < NW3; ++k) sum += act_w[k];
        a.nb[T.tile] = nb_s;
        a.tile_act[T.tile] = static_cast<int32_t>(sum);
    }
}

struct Merge3Args {
    Geo3 g;
    const uint16_t *codes;
    const uint16_t *xface;  // as written by k3_tile
    int32_t *gparent;
};

// Fixed random priority of an id: a bijection of the 32-bit integers
// (multiplications by odd constants and xor-shifts), so no two ids tie.
__device__ __forceinline__ uint32_t id_prio(int x)
{
    uint32_t h = static_cast<uint32_t>(x) * 0x9E3779B1u;
    h ^= h >> 16;
    h *= 0x85EBCA6Bu;
    h ^= h >> 13;
    return h;
}

// Union of the trees holding ids a and b: the root of lower priority is
// linked below the other by a device-scope compare-and-swap (randomised
// linking keeps the expected depth logarithmic); a failed swap returns the
// root's new parent, from which the union goes on.  The walks halve their
// paths as in the square-lattice merge.
__device__ __forceinline__ void gunite_prio(int *G, int a, int b)
{
    gfind2_from<false>(G, a, b, G[a], G[b]);
    for (;;) {
        if (a == b) return;
        if (id_prio(a) > id_prio(b)) {
            const int t = a;
            a = b;
            b = t;
        }
        int expect = a;
        if (__hip_atomic_compare_exchange_strong(&G[a], &expect, b, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return;
        a = expect;
        gfind2_again(G, a, b, true);
    }
}

// Tile consolidation: each active bond leaving the tile through its +x, +y or
// +z face joins the ids of its two ends (both are face sites, hence claimed).
// Every face has one neighbouring tile, so (face, id, id across) names a
// union.  The workgroup first gathers its distinct unions into a list (the
// codes of all its face positions, which carry the bond bits, loaded at once,
// then the codes across the active ones, duplicates dropped), then works the list off with every lane
// busy: a lane no longer waits for its wave's deepest union at each of its
// face positions.
template <int MT>
__global__ __launch_bounds__(MT) void k3_merge(Merge3Args a)
{
    constexpr int MPOS = (FX + FY + FZ + MT - 1) / MT;  // face positions per thread
    // seen[d][h]: the last pair (ca << 16 | cb) registered across face d in
    // hash slot h = ca mod MSEEN; a lane that gets its own pair back skips it
    // (the lane that registered it lists it; pairs sharing a slot are at
    // worst listed twice)
    __shared__ unsigned int seen[3][MSEEN];
    __shared__ unsigned int list[FX + FY + FZ];  // d << 30 | ca << 15 | cb
    __shared__ int nlist;
    const Geo3 g = a.g;
    const TileOf T = tile_of(g, xcd_remap(blockIdx.x, g.ntiles));
    for (int k = threadIdx.x; k < 3 * MSEEN; k += MT) (&seen[0][0])[k] = 0xFFFFFFFFu;
    if (threadIdx.x == 0) nlist = 0;
    // the neighbouring tile across each face
    const int tx = T.gx0 / CX, ty = T.gy0 / CY, tz = T.gz0 / CZ;
    const int nbr[3] = {(tz * g.nty + ty) * g.ntx + (tx + 1 == g.ntx ? 0 : tx + 1),
                        (tz * g.nty + (ty + 1 == g.nty ? 0 : ty + 1)) * g.ntx + tx,
                        ((tz + 1 == g.ntz ? 0 : tz + 1) * g.nty + ty) * g.ntx + tx};
    // face position f: its direction, and the positions of its site's code and
    // of the code across the face; false outside a ragged tile
    auto face = [&](int f, int &d, int &s1, int &s2) -> bool {
        int lx, ly, lz;
        if (f < FX) {
            d = 0;
            lx = T.tw - 1;
            ly = f % CY;
            lz = f / CY;
            s1 = FX + f;  // in the packed x faces
            s2 = f;
        } else if (f < FX + FY) {
            d = 1;
            lx = (f - FX) % CX;
            ly = T.th - 1;
            lz = (f - FX) / CX;
            s1 = code_pos(lx, ly, lz);
            s2 = code_pos(lx, 0, lz);
        } else {
            d = 2;
            lx = (f - FX - FY) % CX;
            ly = (f - FX - FY) / CX;
            lz = T.td - 1;
            s1 = code_pos(lx, ly, lz);
            s2 = code_pos(lx, ly, 0);
        }
        return f < FX + FY + FZ && lx < T.tw && ly < T.th && lz < T.td;
    };
    int ca[MPOS], cb[MPOS], dd[MPOS];
    bool act[MPOS];
#pragma unroll
    for (int j = 0; j < MPOS; ++j) {  // every own code, its bond bit with it, first (independent loads)
        int s1, s2;
        const int f = j * MT + static_cast<int>(threadIdx.x);
        const bool in = face(f, dd[j], s1, s2);
        uint32_t c = 0;
        if (in)
            c = dd[j] == 0 ? a.xface[static_cast<int64_t>(T.tile) * (2 * FX) + s1]
                           : a.codes[static_cast<int64_t>(T.tile) * CSITES + s1];
        act[j] = ((c >> (dd[j] == 2 ? 14 : 15)) & 1u) != 0u;
        ca[j] = dd[j] == 0 ? static_cast<int>(c & 0x7FFFu) : static_cast<int>(c & CODE_MASK) - CSITES;
        cb[j] = s2;
    }
#pragma unroll
    for (int j = 0; j < MPOS; ++j) {  // then the codes across the active ones
        if (!act[j]) continue;
        if (dd[j] == 0)
            cb[j] = a.xface[static_cast<int64_t>(nbr[0]) * (2 * FX) + cb[j]];
        else
            cb[j] = static_cast<int>(a.codes[static_cast<int64_t>(nbr[dd[j]]) * CSITES + cb[j]] & CODE_MASK) - CSITES;
        if (static_cast<unsigned>(ca[j]) >= CAP || static_cast<unsigned>(cb[j]) >= CAP)
            act[j] = false;  // face sites always hold ids
    }
    __syncthreads();  // seen and nlist are set
#pragma unroll
    for (int j = 0; j < MPOS; ++j) {
        const int pa = __shfl_up(act[j] ? ca[j] : -1, 1), pb = __shfl_up(cb[j], 1), pd = __shfl_up(dd[j], 1);
        bool keep = act[j] && !((threadIdx.x & 63) != 0 && pa == ca[j] && pb == cb[j] && pd == dd[j]);
        if (keep) {
            const unsigned int key = (static_cast<unsigned int>(ca[j]) << 16) | static_cast<unsigned int>(cb[j]);
            keep = atomicExch(&seen[dd[j]][ca[j] % MSEEN], key) != key;
        }
        if (keep)
            list[atomicAdd(&nlist, 1)] = (static_cast<unsigned int>(dd[j]) << 30) |
                                         (static_cast<unsigned int>(ca[j]) << 15) | static_cast<unsigned int>(cb[j]);
    }
    __syncthreads();
    const int n = nlist;
    for (int k = threadIdx.x; k < n; k += MT) {
        const unsigned int e = list[k];
        const int d = static_cast<int>(e >> 30), ia = static_cast<int>((e >> 15) & 0x7FFFu),
                  ib = static_cast<int>(e & 0x7FFFu);
        gunite_prio(a.gparent, T.tile * CAP + ia, nbr[d] * CAP + ib);
    }
}

struct Flat3Args {
    Geo3 g;
    uint8_t *spins;
    int32_t *labels;  // or nullptr
    const uint16_t *codes;
    const int32_t *gkey;     // a root's key: its cluster's minimum site index
    const int32_t *gparent;  // resolved: every id's entry is its root
    const int32_t *nb;
    int32_t *tile_ncl;       // [ntiles]: clusters whose root lies in the tile
    uint32_t q, ising, k0, k1, t, sid;
};

// New state of the cluster whose canonical root is R: word R & 3 of
// block(R >> 2, t, FLIP), as on the square lattice.
__device__ __forceinline__ uint32_t new_state(uint32_t R, const Flat3Args &a)
{
    const U4 b = philox4x32_10(R >> 2, a.t, TAG_FLIP, a.sid, a.k0, a.k1);
    return draw_state(pick(b, R & 3u), a.q);
}

// Every id of every tile resolved after the merge:
// the id's entry is pointed at its root (the trees are final, so concurrent
// walks stay valid) and the id's key (the minimum site index of its part of
// the cluster) is taken into the root's key by an atomic minimum, so that the
// root's key then holds the cluster's minimum site index: its canonical label.
// The ids of one cluster must not all go to its root: a tile first takes the
// minimum per root in a small LDS table (a root whose slot is another's goes to
// memory by itself), and a minimum is only issued if memory's key, read past
// the caches, is larger.  Bound by latency, the walks' and that of a few
// atomics; an atomic an id whose cached key looked larger made it wait for
// one address in the ordered phase (cubic q = 3, K = 0.6: 160^3 47 -> 17 us,
// 512^3 sweep 1320 -> 1022 us).
struct Resolve3Args {
    Geo3 g;
    int32_t *gkey;
    int32_t *gparent;
    const int32_t *nb;
};

template <int RT>
__global__ __launch_bounds__(RT) void k3_resolve(Resolve3Args a)
{
    // a workgroup per tile, its threads over the tile's ids
    constexpr int SLOTS = 256;
    __shared__ int32_t owner[SLOTS], least[SLOTS];
    const int tile = static_cast<int>(blockIdx.x);
    const int nbt = a.nb[tile];
    for (int k = threadIdx.x; k < SLOTS; k += RT) {
        owner[k] = -1;
        least[k] = 0x7FFFFFFF;
    }
    __syncthreads();
    auto take = [&](int root, int32_t key) {
        const int32_t now = __hip_atomic_load(&a.gkey[root], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (key < now) atomicMin(&a.gkey[root], key);
    };
    for (int k = threadIdx.x; k < nbt; k += RT) {
        const int id = tile * CAP + k;
        const int32_t key = a.gkey[id];  // a root's key is not used; another id's never changes
        int x = id, p = a.gparent[x];
        while (p != x) {
            x = p;
            p = a.gparent[x];
        }
        if (x == id) continue;
        a.gparent[id] = x;
        const int h = static_cast<int>((static_cast<uint32_t>(x) * 0x9E3779B1u) >> 24);
        const int was = atomicCAS(&owner[h], -1, x);
        if (was == -1 || was == x)
            atomicMin(&least[h], key);
        else
            take(x, key);
    }
    __syncthreads();
    for (int k = threadIdx.x; k < SLOTS; k += RT)
        if (owner[k] >= 0) take(owner[k], least[k]);
}

// LABEL: labels only (no draws, spins untouched).
// FOUR (Lx a multiple of 4): about a third of the sites of a critical lattice
// are roots, so every site draws, a block of four words for the four sites of a
// lane pair (the even lane for one row, the odd one for the next, as the tile
// kernel's +z words), and a root's state is where its cluster's sites look it
// up, its own slot; the other slots' states are not read.  Otherwise the
// interior roots are listed and draw 64 at a time.  Bound by the ids' scattered
// keys and VALU issue (busy 0.63); 512^3 at beta_c, listed -> all: 213 -> 201 us.
template <bool LABEL, bool FOUR>
__global__ __launch_bounds__(NT3) void k3_flatten(Flat3Args a)
{
    constexpr uint32_t NCODE = CSITES + CAP;
    constexpr bool LIST = !LABEL && !FOUR;
    __shared__ alignas(4) uint8_t ST[LABEL ? 1 : NCODE];  // new state per code (written in pairs)
    __shared__ int32_t Rb[CAP];                   // canonical label per id (labels only)
    __shared__ uint16_t roots[LIST ? NW3 : 1][LIST ? 128 * ITER : 1];  // interior root slots of each wave's rows
    __shared__ unsigned ncl_w[NW3];
    const Geo3 g = a.g;
    const TileOf T = tile_of(g, xcd_remap(blockIdx.x, g.ntiles));
    const int lane = threadIdx.x & 63, w = wave_id();
    // the tile kernel's lanes: two sites of plane lz, rows ly0 ...
    const int lx0 = 2 * (lane % LPR), lz = (w >> 1) * SUB + lane / LPR, ly0 = (w & 1) * ITER;
    const int nr = max(0, min(ITER, T.th - ly0));
    const bool v0 = lz < T.td && lx0 < T.tw, v1 = lz < T.td && lx0 + 1 < T.tw;
    const int nbt = a.nb[T.tile];
    // the lane's codes (two per step), loaded ahead of the ids' chains
    const uint32_t *codes32 = reinterpret_cast<const uint32_t *>(a.codes + static_cast<int64_t>(T.tile) * CSITES) +
                              w * ITER * 64 + lane;
    uint32_t cc[ITER];
#pragma unroll
    for (int it = 0; it < ITER; ++it) cc[it] = it < nr ? codes32[it * 64] & (CODE_MASK | CODE_MASK << 16) : 0u;
    unsigned nbroot = 0;
    for (int k = threadIdx.x; k < nbt; k += NT3) {
        const int id = T.tile * CAP + k;
        const int r = a.gparent[id];  // resolved: the entry is the root
        const int32_t key = a.gkey[r];
        if constexpr (!LABEL) ST[CSITES + k] = static_cast<uint8_t>(new_state(static_cast<uint32_t>(key), a));
        if (LABEL || a.labels) Rb[k] = key;
        nbroot += r == id ? 1u : 0u;
    }
    const uint32_t i_first = (static_cast<uint32_t>(T.gz0 + lz) * static_cast<uint32_t>(g.Ly) +
                              static_cast<uint32_t>(T.gy0 + ly0)) * static_cast<uint32_t>(g.Lx) +
                             static_cast<uint32_t>(T.gx0 + lx0);
    const uint64_t in0 = __ballot(v0), in1 = __ballot(v1);
    const int own_first = lz * PLANE + ly0 * CX + lx0;
    const bool odd_lane = (lane & 1) != 0;
    uint32_t next0 = 0, next1 = 0;  // words of the next row's sites, drawn with this one
    int nroot = 0;
    uint16_t *mylist = roots[LIST ? w : 0];
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        if (it >= nr) break;
        const int s = own_first + it * CX;  // interior roots carry their own slot as code
        const EO m = EO{lanes_eq(cc[it] & 0xFFFFu, static_cast<uint32_t>(s)) & in0,
                        lanes_eq(cc[it] >> 16, static_cast<uint32_t>(s + 1)) & in1};
        if constexpr (LIST) {
            eo_append(mylist, nroot, m, s, s + 1);
        } else {
            nroot += __popcll(m.e) + __popcll(m.o);
            if constexpr (!LABEL) {
                uint32_t w0 = next0, w1 = next1;
                if ((it & 1) == 0) {
                    const uint32_t i0 = i_first + static_cast<uint32_t>(it) * static_cast<uint32_t>(g.Lx);
                    const uint32_t four = odd_lane ? i0 - 2u + static_cast<uint32_t>(g.Lx) : i0;
                    const U4 f = philox4x32_10(four >> 2, a.t, TAG_FLIP, a.sid, a.k0, a.k1);
                    const uint32_t ra = swap_pair_lanes(odd_lane ? f.v0 : f.v2);
                    const uint32_t rb = swap_pair_lanes(odd_lane ? f.v1 : f.v3);
                    w0 = odd_lane ? ra : f.v0;
                    w1 = odd_lane ? rb : f.v1;
                    next0 = odd_lane ? f.v2 : ra;
                    next1 = odd_lane ? f.v3 : rb;
                }
                *reinterpret_cast<uint16_t *>(&ST[s]) =
                    static_cast<uint16_t>(draw_state(w0, a.q) | (draw_state(w1, a.q) << 8));
            }
        }
    }
    if constexpr (LIST) {
        wave_lds_fence();
        for (int k = lane; k < nroot; k += 64) {
            const int s = mylist[k];
            ST[s] = static_cast<uint8_t>(new_state(static_cast<uint32_t>(site_of(g, T, s)), a));
        }
    }
    __syncthreads();
    const bool even_lx = FOUR || (g.Lx & 1) == 0;  // every row starts even: both sites in one store
#pragma unroll
    for (int it = 0; it < ITER; ++it) {
        if (it >= nr) break;
        const uint32_t i0 = i_first + static_cast<uint32_t>(it) * static_cast<uint32_t>(g.Lx);
        const uint32_t c0 = cc[it] & 0xFFFFu, c1 = cc[it] >> 16;
        if constexpr (!LABEL) {
            // (the sites outside a ragged tile carry some code: looked up
            // inside the table, never stored)
            const uint32_t st0 = ST[min(c0, NCODE - 1u)], st1 = ST[min(c1, NCODE - 1u)];
            const uint32_t b0 = a.ising ? (2u * st0 - 1u) & 0xFFu : st0, b1 = a.ising ? (2u * st1 - 1u) & 0xFFu : st1;
            if (even_lx) {
                if (v1) *reinterpret_cast<uint16_t *>(a.spins + i0) = static_cast<uint16_t>(b0 | (b1 << 8));
            } else {
                if (v0) a.spins[i0] = static_cast<uint8_t>(b0);
                if (v1) a.spins[i0 + 1] = static_cast<uint8_t>(b1);
            }
        }
        if (a.labels) {
            auto label = [&](uint32_t c) {
                return c >= static_cast<uint32_t>(CSITES) ? Rb[min(c, NCODE - 1u) - CSITES]
                                                          : site_of(g, T, static_cast<int>(c));
            };
            const int32_t R0 = label(c0), R1 = label(c1);
            if (even_lx) {
                if (v1) *reinterpret_cast<int2 *>(a.labels + i0) = make_int2(R0, R1);
            } else {
                if (v0) a.labels[i0] = R0;
                if (v1) a.labels[i0 + 1] = R1;
            }
        }
    }
    const unsigned long long tot = wave_sum(nbroot);
    if (lane == 0) ncl_w[w] = static_cast<unsigned>(tot) + static_cast<unsigned>(nroot);
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned sum = 0;
        for (int k = 0; k < NW3; ++k) sum += ncl_w[k];
        a.tile_ncl[T.tile] = static_cast<int32_t>(sum);
    }
}

// The cluster count of a labeling from the tiles' counts, by one workgroup.
__global__ __launch_bounds__(1024) void k3_count_out(const int32_t *tile_ncl, int ntiles, int32_t *n_clusters)
{
    sum_tiles(tile_ncl, ntiles, n_clusters);
}

}  // namespace cubic
}  // namespace swccl

using namespace swccl;
using namespace swccl::cubic;

namespace {

constexpr size_t ALIGN3 = 256;
// Up to this many tiles the tile kernel takes 16 waves a tile, four steps each,
// else 8 of eight: a wave's steps follow each other, and there are waves to spare.
// Critical Ising sweep, 8 -> 16 waves: 100 x 75 x 61 (80 tiles) 51.3 -> 45.8 us,
// 101 x 75 x 61 59.0 -> 51.5, 160^3 (500) 71.2 -> 67.4; 192 x 192 x 176 (792) 96.5 ->
// 97.7, 200 x 210 x 200 (1274) 122.8 -> 122.7, 256 x 256 x 192 (1536) 133 -> 137, 256^3
// 159 -> 166, and in the ordered phase (q = 3, K = 0.6) 117 -> 119, 140 -> 144, 162 ->
// 167, 193 -> 203.
constexpr int TILE3_SMALL = 512;
// Up to this many tiles the merge takes 1024 threads a tile, else 256.  Critical
// Ising sweep, 256 -> 1024: 100 x 75 x 61 (80 tiles) 55.5 -> 51.6 us, 160^3 (500)
// 75 -> 72, 256^3 (2048) 161 -> 175.
constexpr int MERGE3_WIDE = 512;
// Up to this many tiles the resolve takes 512 threads a tile, else 256.  64 -> 256
// -> 512: 160^3 105 -> 80 -> 75 us, 200 x 210 x 220 (1372 tiles) 163 -> 133 ->
// 132, in the ordered phase 220 -> 208 -> 220; 128 or 1024 at 256^3 170, 256 162.
constexpr int RESOLVE3_WIDE = 1024;
size_t up3(size_t v) { return (v + ALIGN3 - 1) / ALIGN3 * ALIGN3; }
int64_t cdiv3(int64_t a, int64_t b) { return (a + b - 1) / b; }

struct Layout3 {
    Geo3 g;
    int64_t N;
    size_t codes, xface, gkey, gparent, nb, tile_act, tile_ncl, ticket, obs_part, total;
};

// Extents >= 1, N < 2^31, and the ids of all tiles (ntiles x CAP) index
// int32 arrays.
sw_status check_shape3(int32_t Lx, int32_t Ly, int32_t Lz)
{
    if (Lx < 1 || Ly < 1 || Lz < 1) return SW_ERR_SIZE;
    const int64_t N = static_cast<int64_t>(Lx) * Ly * Lz;
    if (N >= (static_cast<int64_t>(1) << 31)) return SW_ERR_SIZE;
    const int64_t nt = cdiv3(Lx, CX) * cdiv3(Ly, CY) * cdiv3(Lz, CZ);
    if (nt * CAP >= (static_cast<int64_t>(1) << 31)) return SW_ERR_SIZE;
    return SW_OK;
}

sw_status check3(const sw3_params *p)
{
    if (!p) return SW_ERR_ARG;
    if (p->q < 2 || p->q > 255) return SW_ERR_ARG;
    if (p->spin_kind != SW_SPIN_ISING_I8 && p->spin_kind != SW_SPIN_POTTS_U8) return SW_ERR_ARG;
    if (p->spin_kind == SW_SPIN_ISING_I8 && p->q != 2) return SW_ERR_ARG;
    if (std::isnan(p->K) || p->flags != 0 || p->reserved != 0) return SW_ERR_ARG;
    return check_shape3(p->Lx, p->Ly, p->Lz);
}

// observed: a sweep's workspace, which also holds the observables' ticket and
// partial sums (a labeling takes none).
Layout3 layout3(int32_t Lx, int32_t Ly, int32_t Lz, bool observed)
{
    Layout3 L{};
    L.g.Lx = Lx;
    L.g.Ly = Ly;
    L.g.Lz = Lz;
    L.g.ntx = static_cast<int>(cdiv3(Lx, CX));
    L.g.nty = static_cast<int>(cdiv3(Ly, CY));
    L.g.ntz = static_cast<int>(cdiv3(Lz, CZ));
    L.g.ntiles = L.g.ntx * L.g.nty * L.g.ntz;
    L.N = static_cast<int64_t>(Lx) * Ly * Lz;
    const size_t nt = static_cast<size_t>(L.g.ntiles);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += up3(bytes);
        return at;
    };
    L.codes = take(nt * CSITES * sizeof(uint16_t));
    L.xface = take(nt * 2 * FX * sizeof(uint16_t));
    L.gkey = take(nt * CAP * sizeof(int32_t));
    L.gparent = take(nt * CAP * sizeof(int32_t));
    L.nb = take(nt * sizeof(int32_t));
    L.tile_act = take(nt * sizeof(int32_t));
    L.tile_ncl = take(nt * sizeof(int32_t));
    if (observed) {
        L.ticket = take(sizeof(uint32_t));
        L.obs_part = take(OBS_PART_BYTES);
    }
    L.total = off;
    return L;
}

Layout3 layout3(const sw3_params *p) { return layout3(p->Lx, p->Ly, p->Lz, true); }

template <bool LABEL>
void launch_tile3(const Tile3Args &ta, hipStream_t s)
{
    const dim3 tiles(static_cast<unsigned>(ta.g.ntiles));
    const bool four = ta.g.Lx % 4 == 0;
    if (ta.g.ntiles <= TILE3_SMALL) {
        if (four)
            hipLaunchKernelGGL((k3_tile<LABEL, true, ITER / 2>), tiles, dim3(2 * NT3), 0, s, ta);
        else
            hipLaunchKernelGGL((k3_tile<LABEL, false, ITER / 2>), tiles, dim3(2 * NT3), 0, s, ta);
    } else if (four) {
        hipLaunchKernelGGL((k3_tile<LABEL, true, ITER>), tiles, dim3(NT3), 0, s, ta);
    } else {
        hipLaunchKernelGGL((k3_tile<LABEL, false, ITER>), tiles, dim3(NT3), 0, s, ta);
    }
}

// The merge and the resolve are chains of dependent global accesses: while the
// tiles leave waves to spare, more threads a tile shorten them.
void launch_merge3(const Merge3Args &ma, hipStream_t s)
{
    const dim3 tiles(static_cast<unsigned>(ma.g.ntiles));
    if (ma.g.ntiles <= MERGE3_WIDE)
        hipLaunchKernelGGL(k3_merge<1024>, tiles, dim3(1024), 0, s, ma);
    else
        hipLaunchKernelGGL(k3_merge<256>, tiles, dim3(256), 0, s, ma);
}

void launch_resolve3(const Resolve3Args &ra, hipStream_t s)
{
    const dim3 tiles(static_cast<unsigned>(ra.g.ntiles));
    if (ra.g.ntiles <= RESOLVE3_WIDE)
        hipLaunchKernelGGL(k3_resolve<512>, tiles, dim3(512), 0, s, ra);
    else
        hipLaunchKernelGGL(k3_resolve<256>, tiles, dim3(256), 0, s, ra);
}

template <bool LABEL>
void launch_flatten3(const Flat3Args &fa, hipStream_t s)
{
    const dim3 tiles(static_cast<unsigned>(fa.g.ntiles));
    if (fa.g.Lx % 4 == 0)
        hipLaunchKernelGGL((k3_flatten<LABEL, true>), tiles, dim3(NT3), 0, s, fa);
    else
        hipLaunchKernelGGL((k3_flatten<LABEL, false>), tiles, dim3(NT3), 0, s, fa);
}

template <typename T>
T *at3(void *ws, size_t off)
{
    return reinterpret_cast<T *>(static_cast<char *>(ws) + off);
}

}  // namespace

extern "C" {

size_t sw3_workspace_bytes(const sw3_params *p)
{
    if (check3(p) != SW_OK) return 0;
    return layout3(p).total;
}

sw_status sw3_init_spins(const sw3_params *p, uint8_t *spins, void *stream)
{
    const sw_status st = check3(p);
    if (st != SW_OK) return st;
    if (!spins) return SW_ERR_ARG;
    const int64_t N = static_cast<int64_t>(p->Lx) * p->Ly * p->Lz;
    return swccl_internal::init_spins(spins, N, p->q, p->spin_kind == SW_SPIN_ISING_I8, p->seed, p->stream_id,
                                      static_cast<hipStream_t>(stream));
}

size_t ccl3_workspace_bytes(int32_t Lx, int32_t Ly, int32_t Lz)
{
    if (check_shape3(Lx, Ly, Lz) != SW_OK) return 0;
    return layout3(Lx, Ly, Lz, false).total;
}

sw_status ccl3_label(const uint8_t *bonds, int32_t Lx, int32_t Ly, int32_t Lz, int32_t *labels, int32_t *n_clusters,
                     void *workspace, size_t workspace_bytes, void *stream)
{
    const sw_status st = check_shape3(Lx, Ly, Lz);
    if (st != SW_OK) return st;
    if (!bonds || !labels) return SW_ERR_ARG;
    const Layout3 L = layout3(Lx, Ly, Lz, false);
    if (!workspace || workspace_bytes < L.total || reinterpret_cast<uintptr_t>(workspace) % ALIGN3)
        return SW_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    Tile3Args ta{};
    ta.g = L.g;
    ta.in = bonds;
    ta.codes = at3<uint16_t>(workspace, L.codes);
    ta.xface = at3<uint16_t>(workspace, L.xface);
    ta.gkey = at3<int32_t>(workspace, L.gkey);
    ta.gparent = at3<int32_t>(workspace, L.gparent);
    ta.nb = at3<int32_t>(workspace, L.nb);
    ta.tile_act = at3<int32_t>(workspace, L.tile_act);
    ta.tany = 1u;
    Merge3Args ma{};
    ma.g = L.g;
    ma.codes = ta.codes;
    ma.xface = ta.xface;
    ma.gparent = ta.gparent;
    Resolve3Args ra{};
    ra.g = L.g;
    ra.gkey = ta.gkey;
    ra.gparent = ta.gparent;
    ra.nb = ta.nb;
    Flat3Args fa{};
    fa.g = L.g;
    fa.labels = labels;
    fa.codes = ta.codes;
    fa.gkey = ta.gkey;
    fa.gparent = ta.gparent;
    fa.nb = ta.nb;
    fa.tile_ncl = at3<int32_t>(workspace, L.tile_ncl);
    launch_tile3<true>(ta, s);
    launch_merge3(ma, s);
    launch_resolve3(ra, s);
    launch_flatten3<true>(fa, s);
    if (n_clusters) hipLaunchKernelGGL(k3_count_out, dim3(1), dim3(1024), 0, s, fa.tile_ncl, L.g.ntiles, n_clusters);
    return swccl_internal::device_error(hipGetLastError(), "ccl3_label");
}

sw_status sw3_sweep(const sw3_params *p, uint8_t *spins, uint32_t t0, int32_t n, uint8_t *bonds, int32_t *labels,
                    int64_t *records, void *workspace, size_t workspace_bytes, void *stream)
{
    const sw_status st = check3(p);
    if (st != SW_OK) return st;
    if (!spins || n < 0) return SW_ERR_ARG;
    if (static_cast<uint64_t>(t0) + static_cast<uint64_t>(n) > (static_cast<uint64_t>(1) << 32)) return SW_ERR_STATE;
    const Layout3 L = layout3(p);
    if (!workspace || workspace_bytes < L.total || reinterpret_cast<uintptr_t>(workspace) % ALIGN3)
        return SW_ERR_WORKSPACE;
    if (n == 0) return SW_OK;
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint64_t T = swccl_internal::bond_threshold(p->K);

    Tile3Args ta{};
    ta.g = L.g;
    ta.in = spins;
    ta.bonds = bonds;
    ta.codes = at3<uint16_t>(workspace, L.codes);
    ta.xface = at3<uint16_t>(workspace, L.xface);
    ta.gkey = at3<int32_t>(workspace, L.gkey);
    ta.gparent = at3<int32_t>(workspace, L.gparent);
    ta.nb = at3<int32_t>(workspace, L.nb);
    ta.tile_act = at3<int32_t>(workspace, L.tile_act);
    ta.tany = T > 0 ? 1u : 0u;
    ta.tm1 = T > 0 ? static_cast<uint32_t>(T - 1) : 0u;
    ta.k0 = static_cast<uint32_t>(p->seed);
    ta.k1 = static_cast<uint32_t>(p->seed >> 32);
    ta.sid = p->stream_id;
    if (records) ta.ticket = at3<uint32_t>(workspace, L.ticket);

    Merge3Args ma{};
    ma.g = L.g;
    ma.codes = ta.codes;
    ma.xface = ta.xface;
    ma.gparent = ta.gparent;

    Flat3Args fa{};
    fa.g = L.g;
    fa.spins = spins;
    fa.codes = ta.codes;
    fa.gkey = ta.gkey;
    fa.gparent = ta.gparent;
    fa.nb = ta.nb;
    fa.tile_ncl = at3<int32_t>(workspace, L.tile_ncl);
    fa.q = static_cast<uint32_t>(p->q);
    fa.ising = p->spin_kind == SW_SPIN_ISING_I8 ? 1u : 0u;
    fa.k0 = ta.k0;
    fa.k1 = ta.k1;
    fa.sid = ta.sid;

    Resolve3Args ra{};
    ra.g = L.g;
    ra.gkey = ta.gkey;
    ra.gparent = ta.gparent;
    ra.nb = ta.nb;

    ObsArgs oa{};
    oa.spins = spins;
    oa.Lx = static_cast<uint32_t>(L.g.Lx);
    oa.Ly = static_cast<uint32_t>(L.g.Ly);
    oa.Lz = static_cast<uint32_t>(L.g.Lz);
    oa.tile_act = ta.tile_act;
    oa.tile_ncl = fa.tile_ncl;
    oa.ntiles = L.g.ntiles;
    oa.part = at3<uint32_t>(workspace, L.obs_part);
    oa.ticket = ta.ticket;
    for (int32_t k = 0; k < n; ++k) {
        const uint32_t t = t0 + static_cast<uint32_t>(k);
        ta.t = t;
        fa.t = t;
        fa.labels = k + 1 == n ? labels : nullptr;
        launch_tile3<false>(ta, s);
        launch_merge3(ma, s);
        launch_resolve3(ra, s);
        launch_flatten3<false>(fa, s);
        if (records) {
            oa.out = records + static_cast<int64_t>(k) * SW3_REC_LEN;
            launch_observe<true, OBS_RECORD3>(oa, fa.ising != 0, s);
        }
    }
    return swccl_internal::device_error(hipGetLastError(), "sw3_sweep");
}

}  // extern "C"

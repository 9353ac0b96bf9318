// uf.hpp -- device helpers shared by the square- and cubic-lattice kernels:
// XCD-aware workgroup placement, lane masks, the lock-free union-find in LDS
// (Sec. II.B.2) and the global union-find over boundary ids (Sec. II.C), wave
// reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace swccl {

// Workgroups are dealt round-robin to the 8 XCDs.  Give each XCD one
// contiguous range of tiles so that tiles sharing halo lines share an L2.
__device__ __forceinline__ int xcd_remap(int b, int n)
{
    const int xcd = b & 7, local = b >> 3;
    const int q = n >> 3, r = n & 7;
    return xcd * q + min(xcd, r) + local;
}

// Bit `lane` of a wave-uniform mask m, for the calling lane: the mask is used
// as the lane condition directly (no per-lane shift).
__device__ __forceinline__ bool lane_bit(uint64_t m, int lane)
{
    (void)lane;
    return __builtin_amdgcn_inverse_ballot_w64(m);
}


// Lane masks: bit L describes lane L (uicmp yields the mask of one compare).
constexpr int CMP_EQ = 32, CMP_NE = 33, CMP_ULT = 36, CMP_ULE = 37;
__device__ __forceinline__ uint64_t lanes_eq(uint32_t x, uint32_t y) { return __builtin_amdgcn_uicmp(x, y, CMP_EQ); }
__device__ __forceinline__ uint64_t lanes_ne(uint32_t x, uint32_t y) { return __builtin_amdgcn_uicmp(x, y, CMP_NE); }
__device__ __forceinline__ uint64_t lanes_lt(uint32_t x, uint32_t y) { return __builtin_amdgcn_uicmp(x, y, CMP_ULT); }
__device__ __forceinline__ uint64_t lanes_le(uint32_t x, uint32_t y) { return __builtin_amdgcn_uicmp(x, y, CMP_ULE); }

// A tile row as two wave ballots: lane L owns sites 2L and 2L+1, bit L of `e`
// belongs to site 2L and bit L of `o` to site 2L+1.  The masks stay in scalar
// registers; the natural-order shift s -> s+1 is (o << 1, e).
struct EO {
    uint64_t e, o;
};

__device__ __forceinline__ EO eo_andnot(EO a, EO b) { return EO{a.e & ~b.e, a.o & ~b.o}; }

// Set bits of m at lanes below the calling lane.
__device__ __forceinline__ int lanes_below(uint64_t m)
{
    return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(m >> 32),
                                                      __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(m), 0u)));
}

// Append the calling lanes' entries to a wave list: ve for the lanes of m.e,
// then vo for those of m.o (the order does not matter); n is the wave-uniform
// list length.
__device__ __forceinline__ void eo_append(uint16_t *list, int &n, EO m, int ve, int vo)
{
    const auto at = [](uint64_t mask, int from) {
        return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                                          __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask),
                                                                                    static_cast<uint32_t>(from))));
    };
    const int pe = at(m.e, n);
    n += __popcll(m.e);
    const int po = at(m.o, n);
    n += __popcll(m.o);
    if (lane_bit(m.e, 0)) list[pe] = static_cast<uint16_t>(ve);
    if (lane_bit(m.o, 0)) list[po] = static_cast<uint16_t>(vo);
}

// Value of x held by the next lane (DPP wave shift; the last lane gets 0).
__device__ __forceinline__ uint32_t from_next_lane(uint32_t x)
{
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(x), 0x130, 0xF, 0xF, false));
}

// The same, the last lane getting `last` (wave-uniform).
__device__ __forceinline__ uint32_t from_next_lane_or(uint32_t x, int last)
{
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(last, static_cast<int>(x), 0x130, 0xF, 0xF, false));
}

// ---- LDS union-find (workgroup scope) ----
__device__ __forceinline__ int lds_ld(int *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_st(int *p, int v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A node's value is the byte offset of its entry (4 x index): directly an LDS
// address.
__device__ __forceinline__ int *lds_entry(int *P, int v)
{
    return reinterpret_cast<int *>(reinterpret_cast<char *>(P) + v);
}

// One step of a union of the trees holding a and b, with a straight-line body
// (nested find/link loops cost more in exec-mask bookkeeping than in LDS
// traffic).  A step climbs both nodes two levels (parent, then grandparent);
// when both are roots the larger is linked below the smaller with an atomic
// min, so every root is the minimum (local, hence global) index of its tree.
// If the larger root had meanwhile been linked elsewhere, the min leaves it
// below its old parent or below the smaller root, and the union goes on with
// that old parent, so no link is lost and every parent stays below its child.
// done is set when the two trees are one.  A lane with nothing to link spends
// its atomic on path halving: min(P[a], grandparent of a) points a at an
// ancestor (entries only ever decrease), which is a no-op when a or its
// parent is a root, so every lane issues the atomic and the step needs no
// branch; the halving keeps the trees shallow for later steps and for the
// compression that follows the unions.  A union also ends when both nodes have
// the same parent, which already makes one tree: a step before both reach the
// root, whose entry every finished lane would otherwise hit.
__device__ __forceinline__ void unite_step(int *P, int &a, int &b, int &done)
{
    const int pa = lds_ld(lds_entry(P, a)), pb = lds_ld(lds_entry(P, b));
    const int ga = lds_ld(lds_entry(P, pa)), gb = lds_ld(lds_entry(P, pb));
    const bool roots = pa == a && pb == b;
    const bool link = roots && a != b;
    const int hi = max(a, b), lo = min(a, b);
    const int old = __hip_atomic_fetch_min(lds_entry(P, link ? hi : a), link ? lo : ga, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
    // bitwise, not short-circuit: the flags stay lane masks (no selects)
    done = static_cast<int>((pa == pb) | (roots & (!link | (old == hi))));
    a = link ? old : ga;
    b = link ? lo : gb;
}

// Root of x (a byte offset, as the tile kernel's parents) once all unions are
// done; a claimed root (negative entry) is a root.
__device__ __forceinline__ int lroot(int *P, int x)
{
    for (;;) {
        const int p = lds_ld(lds_entry(P, x));
        if (p == x || p < 0) return x;
        x = p;
    }
}

// Entries that are done hold FINAL | code << 2 (negative); the entry of an
// unclaimed root, its own byte offset 4 slot, gives its code by the same
// two-bit shift.  P[root] = CLAIMING while a root's id is allocated.
constexpr int CLAIMING = -1;
__device__ __forceinline__ int final_entry(uint32_t code) { return static_cast<int>(0x80000000u | (code << 2)); }
__device__ __forceinline__ uint32_t entry_code(int e) { return (static_cast<uint32_t>(e) >> 2) & 0xFFFFu; }

// Link label x below `up` if x is still a root; returns the entry of x as it
// was: x (linked now), or the parent it has.  The caller knows up < x, so a
// parent stays below its child.
__device__ __forceinline__ int link_root(int *P, int x, int up)
{
    int expect = x;
    __hip_atomic_compare_exchange_strong(lds_entry(P, x), &expect, up, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_WORKGROUP);
    return expect;
}

// ---- global union-find over boundary ids ----
//
// Parents only move towards smaller keys, so a stale (older) parent read from
// a non-coherent L2 is still an ancestor: finds may use plain loads.  Every
// change of a root goes through a device-scope CAS; a failed CAS returns the
// node's current parent, from which the union continues.  Keys are the global
// site indices of the tile-local roots, so every final root's key is the
// minimum site index of its cluster.
__device__ __forceinline__ int gfind(const int *G, int x)
{
    for (;;) {
        const int p = G[x];
        if (p == x) return x;
        x = p;
    }
}

// Parent of x: as this XCD's caches have it (maybe an older one, still an
// ancestor), or FRESH, as it is in memory.
template <bool FRESH>
__device__ __forceinline__ int gparent_of(int *G, int x)
{
    return FRESH ? __hip_atomic_load(&G[x], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : G[x];
}

// Roots of a and b, both chains walked at once (their loads overlap); the
// body is straight-line, a finished chain just reloads its root.  pa and pb are
// the parents of a and b as just read.
template <bool FRESH>
__device__ __forceinline__ void gfind2_from(int *G, int &a, int &b, int pa, int pb)
{
    // path halving: a node passed over is pointed at its grandparent (an
    // ancestor, so concurrent walks stay valid), which keeps the trees of
    // clusters that span many tiles shallow
    while (pa != a || pb != b) {
        const int ga = gparent_of<FRESH>(G, pa), gb = gparent_of<FRESH>(G, pb);
        if (ga != pa) G[a] = ga;
        if (gb != pb) G[b] = gb;
        a = ga;
        b = gb;
        pa = gparent_of<FRESH>(G, a);
        pb = gparent_of<FRESH>(G, b);
    }
}
// The same after a compare-and-swap that failed.  A line cached while its ids
// were roots keeps them roots for this XCD: near a large cluster's root each
// step of a walk on cached parents then ends in another failed swap, so with
// `fresh` the walk reads memory.  Cubic q = 3 sweep in the ordered phase (K =
// 0.6), cached -> fresh: 160^3 111 -> 84 us, 256^3 267 -> 193, 512^3 1055 ->
// 1022, at the critical point within 1%; square q = 3 lattice 8192^2 at 1.4
// beta_c 260 -> 241.  Square lattices of more than MERGE_FRESH_TILES tiles keep
// to the caches: at 16384^2 (32768 tiles) a sweep takes 846 cached, 851 fresh at
// beta_c, 909 and 920 at 1.1 beta_c, 874 and 874 at 1.4, 849 and 846 at 2.0, bond
// percolation 908 and 913 at p = 0.5, 964 and 983 at 0.55, 966 and 953 at 0.7.
// The true crossing lies between: at 11520^2 (16200 tiles) fresh walks would take
// 437 for 436 at beta_c, 490 -> 480 at 1.1, 470 -> 460 at 1.4, and percolation at
// 0.55 556 -> 509.
constexpr int MERGE_FRESH_TILES = 8192;
__device__ __forceinline__ void gfind2_again(int *G, int &a, int &b, bool fresh)
{
    if (fresh)
        gfind2_from<true>(G, a, b, gparent_of<true>(G, a), gparent_of<true>(G, b));
    else
        gfind2_from<false>(G, a, b, G[a], G[b]);
}

__device__ __forceinline__ void gunite(int *G, const int *key, int a, int b, bool fresh)
{
    // the keys are read with the parents: most ids are still roots
    const int a0 = a, b0 = b, pa = G[a], pb = G[b];
    int ka = key[a], kb = key[b];
    gfind2_from<false>(G, a, b, pa, pb);
    if (a != a0) ka = key[a];
    if (b != b0) kb = key[b];
    for (;;) {
        if (a == b) return;
        if (ka < kb) {
            const int t = a, k = ka;
            a = b;
            b = t;
            ka = kb;
            kb = k;
        }
        int expect = a;
        if (__hip_atomic_compare_exchange_strong(&G[a], &expect, b, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return;
        a = expect;  // a was linked meanwhile: continue from its parent
        gfind2_again(G, a, b, fresh);
        ka = key[a];
        kb = key[b];
    }
}

__device__ __forceinline__ unsigned long long wave_sum(unsigned long long v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off);
    return v;
}

// The same for 32-bit values, in all lanes: row sums by DPP row shifts, then
// row broadcasts (a read from outside the row, and rows outside a broadcast's
// row mask, add 0).
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t u)
{
    int v = static_cast<int>(u);
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15, rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31, rows 2 and 3
    return static_cast<uint32_t>(__builtin_amdgcn_readlane(v, 63));
}

// Inclusive prefix sums over the lanes (DPP row shifts, then row broadcasts).
__device__ __forceinline__ uint32_t wave_scan_u32(uint32_t u)
{
    int v = static_cast<int>(u);
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
    return static_cast<uint32_t>(v);
}

// Index of the calling wave in its workgroup, as a wave-uniform (scalar)
// value: everything derived from it (rows, row pointers, loop bounds) then
// stays in scalar registers and branches on it need no exec masking.
__device__ __forceinline__ int wave_id()
{
    return __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
}

// Sum of n int32 counters at a 16-byte aligned address, by one workgroup of
// 1024 threads: 16 counters a thread and step, so that even the counters of the
// largest lattices take a few steps (32768 counters, one a thread and step: 14
// us; two launches of 64 workgroups: 9).
__device__ __forceinline__ void sum_tiles(const int32_t *v, int n, int32_t *out)
{
    __shared__ uint32_t red[16];
    uint32_t acc = 0;
    for (int i = 0; i < n; i += 16 * 1024) {
        uint4 x[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int k = i + 4 * (j * 1024 + static_cast<int>(threadIdx.x));
            if (k + 4 <= n) {
                x[j] = *reinterpret_cast<const uint4 *>(v + k);
            } else {
                x[j].x = k < n ? v[k] : 0;
                x[j].y = k + 1 < n ? v[k + 1] : 0;
                x[j].z = k + 2 < n ? v[k + 2] : 0;
                x[j].w = 0;
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) acc += x[j].x + x[j].y + x[j].z + x[j].w;
    }
    acc = wave_sum_u32(acc);
    if ((threadIdx.x & 63) == 0) red[wave_id()] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int w = 0; w < 16; ++w) t += red[w];
        *out = static_cast<int32_t>(t);
    }
}

__device__ __forceinline__ void add_stat(unsigned long long *p, unsigned long long v)
{
    if (v) __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Keep the compiler from moving LDS accesses of one wave across this point
// (the DS unit executes one wave's LDS operations in order).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}

}  // namespace swccl

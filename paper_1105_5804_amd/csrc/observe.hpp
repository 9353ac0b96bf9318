// observe.hpp -- the observables of a lattice's spins (Eq. potts_hamiltonian:
// -H/J is the number of satisfied bonds) together with the last sweep's
// per-tile counters, in one launch; shared by the square and cubic lattices.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "uf.hpp"

namespace swccl {

constexpr int OBS_NT = 512;          // threads of a workgroup
constexpr int OBS_MAX_BLOCKS = 512;  // one partial row per thread of the last workgroup
constexpr int OBS_FIELDS = 16;       // words of a partial row: satisfied, counts[8], active bonds, clusters, unused
constexpr size_t OBS_PART_BYTES = sizeof(uint32_t) * OBS_MAX_BLOCKS * OBS_FIELDS;

// Where the totals go: a square-lattice record (active, clusters, largest
// cluster, satisfied, counts), a cubic record (active, clusters, satisfied,
// counts) or the observable slots (active, clusters, satisfied, slot 3 left
// alone, counts).
enum ObsOut : int { OBS_RECORD = 0, OBS_RECORD3 = 1, OBS_SLOTS = 2 };

struct ObsArgs {
    const uint8_t *spins;
    uint32_t Lx, Ly, Lz;      // Lz = 1 on the square lattice
    uint32_t segs, units;     // 16-site segments of a row, and of all rows
    const int32_t *tile_act, *tile_ncl;
    int32_t ntiles;           // 0: no sweep yet, nothing to add up
    const int32_t *max_size;  // the sweep's largest cluster, or nullptr
    uint32_t *part;           // [OBS_MAX_BLOCKS][OBS_FIELDS]
    uint32_t *ticket;         // workgroups finished; 0 before the launch
    int64_t *out;
};

// 16 consecutive bytes at any address.
__device__ __forceinline__ uint4 load16(const uint8_t *p)
{
    uint4 v;
    __builtin_memcpy(&v, p, 16);
    return v;
}

// Bit 7 of every byte of x that is zero (exactly: no carry crosses a byte).
__device__ __forceinline__ uint32_t zero_bytes(uint32_t x)
{
    return ~(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x) & 0x80808080u;
}

// Satisfied bonds, state counts 0..7, and the sums of the tiles' counters.
// The spins are read once, 16 sites a load (any alignment: the last segment of
// a row starts 16 before its end and leaves out the sites it shares with the
// one before), and compared bytewise, four sites an instruction; each
// workgroup writes one row of partial sums and the last one to finish adds the
// rows up and writes the record.  Bound by latency on small lattices (one
// load, two reductions and the ticket: 6 us on 457500 cubic sites) and by
// issue on large ones.  With a site a lane, byte loads, separate launches that
// clear, add up the two counters and move the record, and ten 64-bit atomics a
// workgroup, a record of the 4096^2 Ising lattice took 57 us (the counting
// alone 39, twice the sweep's flatten), now 13.5: sweep and record 135 -> 103
// us; of the 2049 x 1537 few-cluster sweep 79 -> 56 us, of the 100 x 75 x 61
// cubic sweep 91 -> 77 us.
template <bool CUBIC, bool ISING, int OUT>
__global__ __launch_bounds__(OBS_NT) void k_observe(ObsArgs a)
{
    constexpr int NW = OBS_NT / 64, NF = 11;
    __shared__ uint32_t red[NW][NF];
    __shared__ int last_s;
    const int lane = threadIdx.x & 63, w = wave_id();
    uint32_t f[NF];  // satisfied, counts[8], active, clusters
#pragma unroll
    for (int k = 0; k < NF; ++k) f[k] = 0;
    const uint32_t Lx = a.Lx, Ly = a.Ly;
    const uint32_t step = gridDim.x * OBS_NT;
    const uint32_t first = blockIdx.x * OBS_NT + threadIdx.x;
    // (row, segment) of the thread's units, advanced without divisions
    const uint32_t step_r = step / a.segs, step_s = step - step_r * a.segs;
    const uint32_t step_z = CUBIC ? step_r / Ly : 0u, step_y = CUBIC ? step_r - step_z * Ly : step_r;
    uint32_t row = first / a.segs, seg = first - row * a.segs;
    uint32_t z = CUBIC ? row / Ly : 0u, y = CUBIC ? row - z * Ly : row;
    for (uint32_t u = first; u < a.units; u += step) {
        const uint32_t r = CUBIC ? z * Ly + y : y;
        const uint8_t *p = a.spins + static_cast<size_t>(r) * Lx;
        const uint8_t *py = a.spins + static_cast<size_t>(y + 1u == Ly ? r - y : r + 1u) * Lx;
        const uint8_t *pz = CUBIC ? a.spins + static_cast<size_t>(z + 1u == a.Lz ? y : r + Ly) * Lx : nullptr;
        if (Lx >= 16u) {
            const uint32_t x = min(seg * 16u, Lx - 16u), skip = seg * 16u - x;
            const uint4 v4 = load16(p + x), y4 = load16(py + x);
            const uint4 z4 = CUBIC ? load16(pz + x) : make_uint4(0u, 0u, 0u, 0u);
            const uint32_t nb = p[x + 16u == Lx ? 0u : x + 16u];  // right of the last site
            const uint32_t v[5] = {v4.x, v4.y, v4.z, v4.w, nb};
            const uint32_t dy[4] = {y4.x, y4.y, y4.z, y4.w}, dz[4] = {z4.x, z4.y, z4.z, z4.w};
            uint32_t n1 = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t drop = min(max(static_cast<int>(skip) - 4 * j, 0), 4);
                const uint32_t in = static_cast<uint32_t>(0x80808080ull << (8u * drop));  // sites counted here
                const uint32_t right = (v[j] >> 8) | (v[j + 1] << 24);
                f[0] += __popc(zero_bytes(v[j] ^ right) & in) + __popc(zero_bytes(v[j] ^ dy[j]) & in);
                if constexpr (CUBIC) f[0] += __popc(zero_bytes(v[j] ^ dz[j]) & in);
                if constexpr (ISING) {
                    n1 += __popc(zero_bytes(v[j] ^ 0x01010101u) & in);
                } else {
                    const uint32_t m = zero_bytes(v[j] & 0xF8F8F8F8u) & in;  // states below 8
                    const uint32_t b0 = v[j] << 7, b1 = v[j] << 6, b2 = v[j] << 5;
                    const uint32_t lo = m & ~b2, hi = m & b2;
                    const uint32_t q0 = lo & ~b1, q1 = lo & b1, q2 = hi & ~b1, q3 = hi & b1;
                    f[1] += __popc(q0 & ~b0);
                    f[2] += __popc(q0 & b0);
                    f[3] += __popc(q1 & ~b0);
                    f[4] += __popc(q1 & b0);
                    f[5] += __popc(q2 & ~b0);
                    f[6] += __popc(q2 & b0);
                    f[7] += __popc(q3 & ~b0);
                    f[8] += __popc(q3 & b0);
                }
            }
            if constexpr (ISING) {
                f[2] += n1;
                f[1] += 16u - skip - n1;
            }
        } else {  // rows shorter than a segment: one unit a row
            for (uint32_t x = 0; x < Lx; ++x) {
                const uint32_t s = p[x];
                f[0] += (s == p[x + 1u == Lx ? 0u : x + 1u] ? 1u : 0u) + (s == py[x] ? 1u : 0u);
                if constexpr (CUBIC) f[0] += s == pz[x] ? 1u : 0u;
                const uint32_t st = ISING ? (s == 1u ? 1u : 0u) : s;
#pragma unroll
                for (int k = 0; k < 8; ++k) f[1 + k] += st == static_cast<uint32_t>(k) ? 1u : 0u;
            }
        }
        seg += step_s;
        const uint32_t carry = seg >= a.segs ? 1u : 0u;
        seg -= carry ? a.segs : 0u;
        y += step_y + carry;
        if constexpr (CUBIC) {
            z += step_z;
            if (y >= Ly) {
                y -= Ly;
                z += 1u;
            }
        }
    }
    for (uint32_t t = first; t < static_cast<uint32_t>(a.ntiles); t += step) {
        f[9] += static_cast<uint32_t>(a.tile_act[t]);
        f[10] += static_cast<uint32_t>(a.tile_ncl[t]);
    }
    auto block_sums = [&]() {  // red[w][k]: the waves' sums of f[k]
#pragma unroll
        for (int k = 0; k < NF; ++k) {
            const uint32_t s = wave_sum_u32(f[k]);
            if (lane == 0) red[w][k] = s;
        }
        __syncthreads();
    };
    block_sums();
    // The rows go to and come from the last workgroup past the caches that are
    // not shared between XCDs, by agent-scope accesses, ordered by waiting for
    // the store before the ticket is taken: an agent-scope fence instead writes
    // the whole L2 back in every wave (77 us a launch at 4096^2).
    if (threadIdx.x < NF) {
        // below 2^32: a workgroup takes a whole small lattice or 1/512 of a large one
        uint32_t s = 0;
#pragma unroll
        for (int k = 0; k < NW; ++k) s += red[k][threadIdx.x];
        __hip_atomic_store(&a.part[blockIdx.x * OBS_FIELDS + threadIdx.x], s, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (threadIdx.x == 0)  // (of the wave that stored the row)
        last_s = __hip_atomic_fetch_add(a.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == gridDim.x;
    __syncthreads();
    if (!last_s) return;
    {
        const bool mine = threadIdx.x < gridDim.x;
        uint64_t *row8 = reinterpret_cast<uint64_t *>(a.part + (mine ? threadIdx.x : 0u) * OBS_FIELDS);
#pragma unroll
        for (int k = 0; k < NF; k += 2) {
            const uint64_t two = __hip_atomic_load(&row8[k / 2], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            f[k] = mine ? static_cast<uint32_t>(two) : 0u;
            if (k + 1 < NF) f[k + 1] = mine ? static_cast<uint32_t>(two >> 32) : 0u;
        }
    }
    block_sums();  // (a wave's 64 rows: at most 3/8 of 2^31 bonds)
    if (threadIdx.x < NF) {
        uint64_t s = 0;
#pragma unroll
        for (int k = 0; k < NW; ++k) s += red[k][threadIdx.x];
        const int k = threadIdx.x;
        constexpr int SAT = OUT == OBS_RECORD ? 3 : 2;  // satisfied; the counts follow (after slot 3 in the slots)
        constexpr int CNT = OUT == OBS_RECORD3 ? 3 : 4;
        const int at = k == 0 ? SAT : k < 9 ? CNT + k - 1 : k - 9;
        a.out[at] = static_cast<int64_t>(s);
    }
    if (OUT == OBS_RECORD && threadIdx.x == NF) a.out[2] = a.max_size ? *a.max_size : -1;
}

// Enqueue the observables of a lattice.  Two workgroups of 512 threads per CU
// at most, each thread one segment on lattices of up to 4 million sites.
template <bool CUBIC, int OUT>
inline void launch_observe(ObsArgs a, bool ising, hipStream_t s)
{
    a.segs = (a.Lx + 15u) / 16u;
    a.units = a.segs * a.Ly * a.Lz;
    const uint32_t blocks = (a.units + OBS_NT - 1u) / OBS_NT;
    const dim3 grid(blocks < OBS_MAX_BLOCKS ? blocks : OBS_MAX_BLOCKS), block(OBS_NT);
    if (ising)
        hipLaunchKernelGGL((k_observe<CUBIC, true, OUT>), grid, block, 0, s, a);
    else
        hipLaunchKernelGGL((k_observe<CUBIC, false, OUT>), grid, block, 0, s, a);
}

}  // namespace swccl

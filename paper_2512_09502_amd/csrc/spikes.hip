// Spike exchange through the built maps (the paper's Appendix E example and
// the collective subsection): per-destination packets of one time step on
// the source host, and on the target host the lookup of received map
// positions (L for point-to-point, I for collective groups) into the image's
// row of the source-sorted connections, expanded into (target, delay,
// weight x multiplicity) events.
//
// Packets: each spike contributes one record per (destination, position)
// pair of its source; the records of a destination follow the order of the
// spikes.  That is a counting sort on the destination alone: the spikes are
// cut into tiles, a tile's records are counted per destination, the counts
// (destination-major) are scanned, and each tile places its records.  Nothing
// is sized by the number of records, so there is one wait, at the end.  One
// step of the 32-area share, 1% of its neurons spiking: count 4.8, scan 7.4,
// place 7.0 us (records one lane a spike 31 us, radix sort, copy and two waits
// before); packets and delivery together 202 -> 90 us.
#include <algorithm>

#include "device_common.h"
#include "internal.h"

namespace snnc {
namespace {

constexpr int SNT = 256;

// Where a call's kernels note an entry outside its range, with plain stores
// (any lane, same value): a mapped pinned word that the host reads after the
// stream's wait (cleared by the host before the launches: the previous call
// waited), and a word in device memory for the call's later kernels, which then
// leave the caller's arrays alone.  The latter holds the number of the last
// call with such an entry, so nothing has to clear it.
struct Bad {
    uint32_t* host;
    uint64_t* dev;
    uint64_t call;
    __device__ __forceinline__ void set() const {
        *host = 1u;
        *dev = call;
    }
    __device__ __forceinline__ bool is_set() const { return *dev == call; }
};

Bad new_bad(Ctx& c) {
    if (!c.exchange_bad) {
        c.exchange_bad = dalloc_n<uint64_t>(c, 1);
        HIPCHK(hipMemsetAsync(c.exchange_bad, 0, 8, c.stream));
    }
    *reinterpret_cast<volatile uint32_t*>(c.tot_pin + 2) = 0u;
    return Bad{reinterpret_cast<uint32_t*>(c.tot_pin_dev + 2), c.exchange_bad, ++c.exchange_calls};
}

// destination rank of a list entry: the host itself (point-to-point) or the
// group's rank among the sorted group ids (collective)
__device__ __forceinline__ uint32_t dest_rank(uint32_t v, const int32_t* groups, uint32_t n_groups) {
    if (!groups) return v;
    uint32_t a = 0, b = n_groups;   // lower_bound
    while (a < b) {
        const uint32_t m = (a + b) >> 1;
        if (groups[m] < (int32_t)v) a = m + 1; else b = m;
    }
    return a;
}

// A call's spikes and the send rows they expand into.
struct Spikes {
    const uint32_t* id;
    uint64_t n;
    uint32_t M;              // ids at or beyond it set the error word
    const uint64_t* ptr;     // send rows
    const uint32_t* dest;
    const uint32_t* where;
    const int32_t* groups;   // null: destinations are hosts
    uint32_t n_groups, n_dest;
    const uint32_t* mult;    // null: 1
};

constexpr int REC_STEPS = 4;             // records of a lane in flight
constexpr uint32_t DEST_RANGE = 4096;    // destinations a wave counts at a time (its counters in LDS)

// a wave's LDS operations take effect in program order: only the compiler is held
__device__ __forceinline__ void lds_in_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One wave walks the records of spikes [k0, k1) in order, 64 at a time:
// lane's f(spike, dest, entry, live).  The rows of 64 spikes are laid end to
// end, so short rows leave no lanes idle; row_of (64 words of the wave's LDS)
// holds where each begins.  A spike without a row (its id is not a local
// neuron's) sets *bad, which may be null.
template <class F>
__device__ __forceinline__ void walk_records(const Spikes& sp, uint64_t k0, uint64_t k1, uint32_t* row_of, uint32_t* bad,
                                             F f) {
    const int lane = threadIdx.x & 63;
    for (uint64_t kb = k0; kb < k1; kb += 64) {
        const uint64_t k = kb + lane;
        uint64_t row = 0;
        uint32_t len = 0;
        if (k < k1) {
            const uint32_t s = sp.id[k];
            if (s >= sp.M) {
                if (bad) *bad = 1u;   // any lane may set it
            } else {
                row = sp.ptr[s];
                len = (uint32_t)(sp.ptr[s + 1] - row);
            }
        }
        const uint32_t incl = wave_incl_scan(len);
        const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        lds_in_order();
        row_of[lane] = incl - len;
        lds_in_order();
        for (uint32_t r0 = 0; r0 < total; r0 += 64 * REC_STEPS) {
            uint32_t at[REC_STEPS], d[REC_STEPS];
            uint64_t j[REC_STEPS];
#pragma unroll
            for (int u = 0; u < REC_STEPS; ++u) {
                const uint32_t r = r0 + u * 64 + lane;
                uint32_t a = 0;   // last row that begins at or before r
#pragma unroll
                for (uint32_t h = 32; h; h >>= 1)
                    if (row_of[a + h] <= r) a += h;
                at[u] = a;
                j[u] = __shfl(row, (int)a, 64) + (r - row_of[a]);
                d[u] = r < total ? sp.dest[j[u]] : 0u;
            }
#pragma unroll
            for (int u = 0; u < REC_STEPS; ++u) {
                const bool live = r0 + u * 64 + lane < total;
                f(kb + at[u], live ? dest_rank(d[u], sp.groups, sp.n_groups) : 0u, j[u], live);
            }
        }
    }
}

// cnt[d * n_tiles + tile]: records of the tile for destination d.  One wave a
// tile and range of DEST_RANGE destinations (blockIdx.y).
__global__ __launch_bounds__(64) void k_packet_count(Spikes sp, uint64_t tile, uint32_t n_tiles, uint32_t* cnt,
                                                     Bad bad) {
    extern __shared__ __align__(8) uint32_t lds[];
    __shared__ uint32_t row_of[64], s_bad;
    if (threadIdx.x == 0) s_bad = 0;
    const uint32_t d0 = blockIdx.y * DEST_RANGE;
    const uint32_t nd = min(sp.n_dest - d0, DEST_RANGE);
    for (uint32_t i = threadIdx.x; i < nd; i += 64) lds[i] = 0;
    __syncthreads();
    const uint64_t k0 = blockIdx.x * tile;
    walk_records(sp, k0, min(k0 + tile, sp.n), row_of, &s_bad, [&](uint64_t, uint32_t d, uint64_t, bool live) {
        if (live && d - d0 < nd) atomicAdd(&lds[d - d0], 1u);
    });
    __syncthreads();
    if (threadIdx.x == 0 && s_bad) bad.set();
    for (uint32_t i = threadIdx.x; i < nd; i += 64) cnt[(uint64_t)(d0 + i) * n_tiles + blockIdx.x] = lds[i];
}

// Places one step's records: next[d] is the wave's next free place of
// destination d; lanes with the same destination go in lane order.
template <class T>
__device__ __forceinline__ void place_records(const Spikes& sp, uint32_t d, bool mine, uint32_t d_bits, T* next,
                                              uint64_t k, uint64_t j, uint32_t* pos_out, uint32_t* mult_out) {
    const int lane = threadIdx.x & 63;
    uint64_t peers = __ballot(mine);
    for (uint32_t b = 0; b < d_bits; ++b) {
        const bool one = (d >> b) & 1u;
        const uint64_t m = __ballot(one);
        peers &= one ? m : ~m;
    }
    if (mine) {
        const uint32_t rank = (uint32_t)__popcll(peers & ((1ull << lane) - 1));
        const T base = next[d];
        lds_in_order();
        if (rank == 0) next[d] = base + (T)__popcll(peers);
        const uint64_t o = (uint64_t)base + rank;
        pos_out[o] = sp.where[j];
        mult_out[o] = sp.mult ? sp.mult[k] : 1u;
    }
    lds_in_order();
}

// nothing is written where the records (first[n_dest * n_tiles]) exceed the caller's capacity or a spike has no row
__global__ __launch_bounds__(64) void k_packet_place(Spikes sp, uint64_t tile, uint32_t n_tiles, uint32_t d_bits,
                                                     const uint64_t* first, uint64_t cap, uint64_t* off,
                                                     uint32_t* pos_out, uint32_t* mult_out, Bad bad) {
    extern __shared__ __align__(8) uint64_t next[];
    __shared__ uint32_t row_of[64];
    const uint64_t total = first[(uint64_t)sp.n_dest * n_tiles];
    if ((total > cap) | bad.is_set()) return;   // both words loaded at once
    const uint32_t d0 = blockIdx.y * DEST_RANGE;
    const uint32_t nd = min(sp.n_dest - d0, DEST_RANGE);
    for (uint32_t i = threadIdx.x; i < nd; i += 64) {
        const uint64_t v = first[(uint64_t)(d0 + i) * n_tiles + blockIdx.x];
        next[i] = v;
        if (blockIdx.x == 0) off[d0 + i] = v;
    }
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) off[sp.n_dest] = total;
    __syncthreads();
    const uint64_t k0 = blockIdx.x * tile;
    walk_records(sp, k0, min(k0 + tile, sp.n), row_of, nullptr, [&](uint64_t k, uint32_t d, uint64_t j, bool live) {
        place_records(sp, d - d0, live && d - d0 < nd, d_bits, next, k, j, pos_out, mult_out);
    });
}

// The same in one workgroup, a tile a wave: one launch where there is little to
// do (50 spikes of a collective group: 7.7 us against three launches of 5 - 7).
constexpr int ONE_NT = 1024;
constexpr uint32_t ONE_WAVES = ONE_NT / 64, ONE_DEST_MAX = 512;
constexpr uint64_t ONE_SPIKES_MAX = 1024, ONE_RECORDS_MAX = 16384;   // spikes, spikes x destinations

__global__ __launch_bounds__(ONE_NT) void k_packets_one(Spikes sp, uint32_t d_bits, uint64_t cap, uint64_t* off,
                                                        uint32_t* pos_out, uint32_t* mult_out, uint64_t* total_out,
                                                        Bad bad) {
    extern __shared__ __align__(8) uint32_t lds[];   // [wave][destination]
    __shared__ uint32_t row_of[ONE_WAVES][64], s_bad;
    if (threadIdx.x == 0) s_bad = 0;
    __shared__ uint64_t scratch[ONE_WAVES];
    const uint32_t wave = threadIdx.x >> 6, nd = sp.n_dest;
    for (uint32_t i = threadIdx.x; i < nd * ONE_WAVES; i += ONE_NT) lds[i] = 0;
    __syncthreads();
    uint32_t* mine = lds + wave * nd;
    const uint64_t tile = (sp.n + ONE_WAVES - 1) / ONE_WAVES;
    const uint64_t k0 = min((uint64_t)wave * tile, sp.n), k1 = min(k0 + tile, sp.n);
    walk_records(sp, k0, k1, row_of[wave], &s_bad, [&](uint64_t, uint32_t d, uint64_t, bool live) {
        if (live) atomicAdd(&mine[d], 1u);
    });
    __syncthreads();
    if (s_bad) {   // the same in every thread
        if (threadIdx.x == 0) bad.set();
        return;
    }
    uint64_t sum = 0;
    if (threadIdx.x < nd)
        for (uint32_t w = 0; w < ONE_WAVES; ++w) sum += lds[w * nd + threadIdx.x];
    uint64_t total;
    const uint64_t before = block_excl_scan<ONE_NT, uint64_t>(sum, scratch, &total);
    if (threadIdx.x == 0) *total_out = total;
    if (total > cap) return;
    if (threadIdx.x < nd) {
        off[threadIdx.x] = before;
        uint32_t at = (uint32_t)before;   // at most ONE_RECORDS_MAX
        for (uint32_t w = 0; w < ONE_WAVES; ++w) {
            const uint32_t v = lds[w * nd + threadIdx.x];
            lds[w * nd + threadIdx.x] = at;
            at += v;
        }
    }
    if (threadIdx.x == 0) off[nd] = total;
    __syncthreads();
    walk_records(sp, k0, k1, row_of[wave], nullptr, [&](uint64_t k, uint32_t d, uint64_t j, bool live) {
        place_records(sp, d, live, d_bits, mine, k, j, pos_out, mult_out);
    });
}

// Delivery: image and row of every received entry, and where its events begin
// among those of its LOOK_NT entries; the sums of these blocks are scanned
// afterwards (by this launch where there is one block).
constexpr int LOOK_NT = 1024;

__global__ __launch_bounds__(LOOK_NT) void k_deliver_lookup(
    const uint32_t* grp, const uint32_t* host, const uint32_t* pos, uint64_t n, uint32_t P, uint32_t PL,
    uint32_t n_maps_grp, int kind, const uint64_t* map_off, const int32_t* map_img, const uint64_t* row_ptr,
    const uint64_t* img_first, const uint32_t* img_count, uint32_t M_local, int32_t* image, uint64_t* rb, uint64_t* re,
    uint64_t* in_block, uint64_t* block_sum, uint64_t* total_out, Bad bad) {
    __shared__ uint64_t scratch[LOOK_NT / 64];
    for (uint64_t e0 = (uint64_t)blockIdx.x * LOOK_NT; e0 < n; e0 += (uint64_t)gridDim.x * LOOK_NT) {
        const uint64_t e = e0 + threadIdx.x;
        uint64_t lo = 0, hi = 0;
        if (e < n) {
            const uint32_t h = host[e];
            bool ok = h < P && (kind == 1 || h != PL);
            uint64_t key = h;
            if (kind == 1) {
                const uint32_t g = grp[e];
                ok = ok && g < n_maps_grp;
                key = (uint64_t)g * P + h;
            }
            int32_t img = -1;
            if (ok) {
                const uint64_t a = map_off[key], b = map_off[key + 1];
                if ((uint64_t)pos[e] < b - a) img = map_img[a + pos[e]];
                else ok = false;
            }
            if (!ok) bad.set();
            if (img >= 0 && img_first) {     // image rows kept apart (GPU memory levels 0 and 1)
                lo = img_first[(uint32_t)img - M_local];
                hi = lo + img_count[(uint32_t)img - M_local];
            } else if (img >= 0) {
                lo = row_ptr[img];
                hi = row_ptr[img + 1];
            }
            image[e] = img;
            rb[e] = lo;
            re[e] = hi;
        }
        uint64_t sum;
        const uint64_t before = block_excl_scan<LOOK_NT, uint64_t>(hi - lo, scratch, &sum);
        if (e < n) in_block[e] = before;
        if (threadIdx.x == 0) {
            block_sum[e0 / LOOK_NT] = total_out ? 0 : sum;
            if (total_out) {   // one block
                block_sum[1] = sum;
                *total_out = sum;
            }
        }
    }
}

// Events: a workgroup takes EV_CHUNK of them.  Two waves find the entries of
// its first and last one (64 probes a step); the entries between are brought
// into LDS, where each event finds its own.  Bound by latency at one step's
// sizes (a search of all entries by each event 30 us, this 12), by the 10 B
// read and 10 B written an event beyond.  Nothing is written where the events
// exceed the caller's capacity or an entry lies outside its map.
constexpr uint32_t EV_CHUNK = 1024, EV_ENTRIES = 512;

__global__ __launch_bounds__(SNT) void k_deliver_events(const uint64_t* block_off, const uint64_t* in_block, uint64_t n,
                                                        uint64_t n_blocks, uint64_t cap, const uint64_t* rb,
                                                        const uint32_t* mult, const int32_t* tgt, const uint16_t* delay,
                                                        const float* weight, int32_t* ev_tgt, uint16_t* ev_delay,
                                                        float* ev_weight, Bad bad) {
    __shared__ uint64_t ends[2], begin[EV_ENTRIES], from[EV_ENTRIES];
    __shared__ float times[EV_ENTRIES];
    const uint64_t total = block_off[n_blocks];
    if ((total > cap) | bad.is_set()) return;   // both words loaded at once
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    auto first_event = [&](uint64_t e) { return block_off[e / LOOK_NT] + in_block[e]; };
    for (uint64_t o0 = (uint64_t)blockIdx.x * EV_CHUNK; o0 < total; o0 += (uint64_t)gridDim.x * EV_CHUNK) {
        const uint32_t here = (uint32_t)min(total - o0, (uint64_t)EV_CHUNK);
        if (wave < 2) {   // last entry that begins at or before the chunk's first / last event
            const uint64_t o = wave ? o0 + here - 1 : o0;
            uint64_t a = 0, b = n;
            while (b - a > 1) {
                const uint64_t step = (b - a + 63) / 64;
                const uint64_t e = a + lane * step;
                const uint64_t m = __ballot(e < b && first_event(e) <= o);
                a += (uint64_t)(__popcll(m) - 1) * step;   // lane 0's probe holds
                b = min(a + step, b);
            }
            if (lane == 0) ends[wave] = a;
        }
        __syncthreads();
        const uint64_t ea = ends[0], eb = ends[1];
        const bool staged = eb - ea < EV_ENTRIES;   // otherwise (many empty rows between) each event searches
        if (staged)
            for (uint32_t i = threadIdx.x; i <= (uint32_t)(eb - ea); i += SNT) {
                begin[i] = first_event(ea + i);
                from[i] = rb[ea + i];
                times[i] = mult ? (float)mult[ea + i] : 1.0f;
            }
        __syncthreads();
#pragma unroll
        for (uint32_t u = 0; u < EV_CHUNK / SNT; ++u) {
            const uint32_t r = u * SNT + threadIdx.x;
            if (r < here) {
                const uint64_t o = o0 + r;
                uint64_t c;
                float m;
                if (staged) {
                    uint32_t a = 0, b = (uint32_t)(eb - ea) + 1;
                    while (b - a > 1) {
                        const uint32_t h = (a + b) >> 1;
                        if (begin[h] <= o) a = h; else b = h;
                    }
                    c = from[a] + (o - begin[a]);
                    m = times[a];
                } else {
                    uint64_t a = ea, b = eb + 1;
                    while (b - a > 1) {
                        const uint64_t h = (a + b) >> 1;
                        if (first_event(h) <= o) a = h; else b = h;
                    }
                    c = rb[a] + (o - first_event(a));
                    m = mult ? (float)mult[a] : 1.0f;
                }
                ev_tgt[o] = tgt[c];
                ev_delay[o] = delay[c];
                ev_weight[o] = weight[c] * m;
            }
        }
        __syncthreads();   // before the next chunk's entries
    }
}

// address of a result array for kernels (host-resident arrays through their mapping)
template <class T>
const T* arr(Ctx& c, int32_t id) {
    auto it = c.arrays.find(id);
    if (it == c.arrays.end()) raise(SNNC_ESTATE, "array not available");
    return static_cast<const T*>(it->second.host ? it->second.dev : it->second.p);
}

template <class T>
const T* arr_or_null(Ctx& c, int32_t id) {
    return c.arrays.count(id) ? arr<T>(c, id) : nullptr;
}

uint32_t bits_for_values(uint64_t n_values) {
    uint32_t b = 0;
    while (b < 64 && (n_values > 0 ? (n_values - 1) >> b : 0)) ++b;
    return b;
}

// Packets of tiles of at least 8 spikes, at most max_tiles of them.
void packets_tiled(Ctx& c, const Spikes& sp, uint64_t max_tiles, uint32_t d_bits, uint64_t cap, uint64_t* off,
                   uint32_t* pos_out, uint32_t* mult_out, const Bad& bad) {
    const uint64_t tile = std::max<uint64_t>(8, (sp.n + max_tiles - 1) / max_tiles);
    const uint32_t n_tiles = (uint32_t)((sp.n + tile - 1) / tile), nd = std::min(sp.n_dest, DEST_RANGE);
    const dim3 grid(n_tiles, (sp.n_dest + DEST_RANGE - 1) / DEST_RANGE);
    const uint64_t cells = (uint64_t)n_tiles * sp.n_dest;
    uint32_t* cnt = dalloc_n<uint32_t>(c, cells);
    uint64_t* first = nullptr;
    try {
        first = dalloc_n<uint64_t>(c, cells + 1);
        tstart(c, "spike_records");
        hipLaunchKernelGGL(k_packet_count, grid, dim3(64), nd * 4, c.stream, sp, tile, n_tiles, cnt, bad);
        tstop(c);
        HIPCHK(hipGetLastError());
        scan_u32_u64_to(c, cnt, first, cells, c.tot_pin_dev);
        tstart(c, "spike_packets");
        hipLaunchKernelGGL(k_packet_place, grid, dim3(64), nd * 8, c.stream, sp, tile, n_tiles, d_bits,
                           (const uint64_t*)first, cap, off, pos_out, mult_out, bad);
        tstop(c);
        HIPCHK(hipGetLastError());
        sync(c);
    } catch (...) {
        dfree(c, cnt);
        dfree(c, first);
        throw;
    }
    dfree(c, cnt);
    dfree(c, first);
}

}  // namespace

uint64_t spike_packets(Ctx& c, int kind, const uint32_t* spikes, const uint32_t* mult, uint64_t n, uint64_t* off,
                       uint32_t* pos_out, uint32_t* mult_out, uint64_t cap) {
    if (!c.prepared) raise(SNNC_ESTATE, "spike packets need a prepared network");
    if (kind != 0 && kind != 1) raise(SNNC_EINVAL, "kind must be 0 (point-to-point) or 1 (collective)");
    if (n >= (1ull << 32)) raise(SNNC_EINVAL, "more than 2^32 - 1 spikes");
    const uint32_t M = c.M[c.P_local];
    const uint64_t* ptr = arr<uint64_t>(c, kind == 0 ? SNNC_TP_PTR : SNNC_GQ_PTR);
    const uint32_t* dest = kind == 0 ? arr<uint32_t>(c, SNNC_T_VAL) : reinterpret_cast<const uint32_t*>(arr<int32_t>(c, SNNC_G_VAL));
    const uint32_t* where = arr<uint32_t>(c, kind == 0 ? SNNC_P_VAL : SNNC_Q_VAL);
    const int32_t* groups = kind == 1 ? arr<int32_t>(c, SNNC_GROUPS) : nullptr;
    const uint32_t n_groups = (uint32_t)c.counts[SNNC_GROUPS];
    const uint32_t n_dest = kind == 0 ? c.P : n_groups;
    if (!n) {
        HIPCHK(hipMemsetAsync(off, 0, ((uint64_t)n_dest + 1) * 8, c.stream));
        sync(c);
        return 0;
    }
    const Spikes sp{spikes, n, M, ptr, dest, where, groups, n_groups, n_dest, mult};
    const uint32_t nd = std::min(n_dest, DEST_RANGE);
    const uint32_t d_bits = bits_for_values(nd);
    const Bad bad = new_bad(c);   // its host word and the total are mapped pinned memory: both read after the wait
    if (n_dest == 0 || (n <= ONE_SPIKES_MAX && n_dest <= ONE_DEST_MAX && n * n_dest <= ONE_RECORDS_MAX)) {
        tstart(c, "spike_packets");
        hipLaunchKernelGGL(k_packets_one, dim3(1), dim3(ONE_NT), ONE_WAVES * nd * 4, c.stream, sp, d_bits, cap, off,
                           pos_out, mult_out, c.tot_pin_dev, bad);
        tstop(c);
        HIPCHK(hipGetLastError());
        sync(c);
    } else {
        // no more counts than four times the records to expect, or 2^18: with fewer tiles a wave has more
        // than one batch of 64 spikes to walk.  4,096 destinations, 50,000 spikes of 8 records: 296 us with
        // 2^18 counts, 222 with one a record, 134 with four
        const double expected = (double)n * (double)c.counts[kind == 0 ? SNNC_T_VAL : SNNC_Q_VAL] / std::max(M, 1u);
        const uint64_t max_cells = std::max<uint64_t>(1ull << 18, (uint64_t)(4 * expected));
        uint64_t max_tiles = std::max<uint64_t>(1, std::min<uint64_t>(1024, max_cells / n_dest));
        for (;; max_tiles = std::max<uint64_t>(1, max_tiles / 8)) {
            try {
                packets_tiled(c, sp, max_tiles, d_bits, cap, off, pos_out, mult_out, bad);
                break;
            } catch (const Error& e) {   // no room for the counts: fewer tiles
                if ((e.code != SNNC_EBUDGET && e.code != SNNC_ENOMEM) || max_tiles == 1) throw;
            }
        }
    }
    if (*reinterpret_cast<volatile uint32_t*>(c.tot_pin + 2)) raise(SNNC_EINVAL, "spike id is not a local neuron");
    return *reinterpret_cast<volatile uint64_t*>(c.tot_pin);   // above cap: the caller reports the small capacity
}

uint64_t deliver(Ctx& c, int kind, const uint32_t* grp, const uint32_t* host, const uint32_t* pos,
                 const uint32_t* mult, uint64_t n, int32_t* image, uint64_t* rb, uint64_t* re, int32_t* ev_tgt,
                 uint16_t* ev_delay, float* ev_weight, uint64_t ev_cap, bool* too_small) {
    if (!c.prepared) raise(SNNC_ESTATE, "delivery needs a prepared network");
    if (kind != 0 && kind != 1) raise(SNNC_EINVAL, "kind must be 0 (point-to-point) or 1 (collective)");
    if (kind == 1 && !grp) raise(SNNC_EINVAL, "collective delivery needs the group ranks");
    *too_small = false;
    const uint64_t* map_off = arr<uint64_t>(c, kind == 0 ? SNNC_R_OFF : SNNC_H_OFF);
    const int32_t* map_img = arr<int32_t>(c, kind == 0 ? SNNC_L_VAL : SNNC_I_VAL);
    const uint64_t* row_ptr = arr<uint64_t>(c, SNNC_ROW_PTR);
    if (!n) {
        sync(c);
        return 0;
    }
    const uint64_t n_blocks = (n + LOOK_NT - 1) / LOOK_NT;
    const bool one = n_blocks == 1;
    const Bad bad = new_bad(c);   // its host word and the total are mapped pinned memory: both read after the wait
    uint64_t* in_block = dalloc_n<uint64_t>(c, n);
    uint64_t *sums = nullptr, *block_off = nullptr;
    try {
        block_off = dalloc_n<uint64_t>(c, n_blocks + 1);
        sums = one ? block_off : dalloc_n<uint64_t>(c, n_blocks);
        tstart(c, "deliver_lookup");
        hipLaunchKernelGGL(k_deliver_lookup, dim3((unsigned)std::min<uint64_t>(n_blocks, 1u << 20)), dim3(LOOK_NT), 0,
                           c.stream, grp, host, pos, n, c.P, c.P_local, (uint32_t)c.counts[SNNC_GROUPS], kind, map_off,
                           map_img, row_ptr, arr_or_null<uint64_t>(c, SNNC_IMG_FIRST),
                           arr_or_null<uint32_t>(c, SNNC_IMG_COUNT), c.M[c.P_local], image, rb, re, in_block, sums,
                           one ? c.tot_pin_dev : (uint64_t*)nullptr, bad);
        tstop(c);
        HIPCHK(hipGetLastError());
        if (!one) scan_u64_u64_to(c, sums, block_off, n_blocks, c.tot_pin_dev);
        if (ev_tgt && ev_cap) {
            // enough workgroups to fill the card; they leave at once where the total is smaller
            const uint64_t chunks = (ev_cap + EV_CHUNK - 1) / EV_CHUNK;
            tstart(c, "deliver_events");
            hipLaunchKernelGGL(k_deliver_events, dim3((unsigned)std::min<uint64_t>(chunks, (uint64_t)c.n_cu * 8)),
                               dim3(SNT), 0, c.stream, (const uint64_t*)block_off, (const uint64_t*)in_block, n, n_blocks,
                               ev_cap, (const uint64_t*)rb, mult, arr<int32_t>(c, SNNC_TGT),
                               arr<uint16_t>(c, SNNC_DELAY), arr<float>(c, SNNC_WEIGHT), ev_tgt, ev_delay, ev_weight, bad);
            tstop(c);
            HIPCHK(hipGetLastError());
        }
        sync(c);
    } catch (...) {
        dfree(c, in_block);
        if (!one) dfree(c, sums);
        dfree(c, block_off);
        throw;
    }
    dfree(c, in_block);
    if (!one) dfree(c, sums);
    dfree(c, block_off);
    if (*reinterpret_cast<volatile uint32_t*>(c.tot_pin + 2)) raise(SNNC_EINVAL, "received entry outside its map");
    const uint64_t total = *reinterpret_cast<volatile uint64_t*>(c.tot_pin);
    *too_small = ev_tgt && total > ev_cap;
    return total;
}

}  // namespace snnc

extern "C" snnc_status snnc_spike_packets(snnc_ctx* ctx, int32_t kind, const uint32_t* spikes, const uint32_t* mult,
                                          uint64_t n, uint64_t* off, uint32_t* pos_out, uint32_t* mult_out,
                                          uint64_t cap, uint64_t* n_out) {
    using namespace snnc;
    if (!ctx || !n_out || (n && !spikes) || !off) return SNNC_EINVAL;
    try {
        HIPCHK(hipSetDevice(ctx->device));
        const uint64_t total = spike_packets(*ctx, kind, spikes, mult, n, off, pos_out, mult_out, cap);
        *n_out = total;
        if (total > cap) {
            ctx->last_error = "packet capacity " + std::to_string(cap) + " below " + std::to_string(total) + " entries";
            return SNNC_EINVAL;
        }
        return SNNC_OK;
    } catch (const Error& e) {
        ctx->last_error = e.msg;
        return e.code;
    }
}

extern "C" snnc_status snnc_deliver(snnc_ctx* ctx, int32_t kind, const uint32_t* grp, const uint32_t* host,
                                    const uint32_t* pos, const uint32_t* mult, uint64_t n, int32_t* image,
                                    uint64_t* row_begin, uint64_t* row_end, int32_t* ev_tgt, uint16_t* ev_delay,
                                    float* ev_weight, uint64_t ev_cap, uint64_t* n_events) {
    using namespace snnc;
    if (!ctx || !n_events || (n && (!host || !pos || !image || !row_begin || !row_end))) return SNNC_EINVAL;
    if (ev_tgt && (!ev_delay || !ev_weight)) return SNNC_EINVAL;
    try {
        HIPCHK(hipSetDevice(ctx->device));
        bool small = false;
        const uint64_t total = deliver(*ctx, kind, grp, host, pos, mult, n, image, row_begin, row_end, ev_tgt,
                                       ev_delay, ev_weight, ev_cap, &small);
        *n_events = total;
        if (small) {
            ctx->last_error = "event capacity " + std::to_string(ev_cap) + " below " + std::to_string(total);
            return SNNC_EINVAL;
        }
        return SNNC_OK;
    } catch (const Error& e) {
        ctx->last_error = e.msg;
        return e.code;
    }
}

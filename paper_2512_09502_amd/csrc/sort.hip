// Stable LSD radix sort of 64-bit keys with a 32-bit payload, one pass per
// digit of at most 9 bits, in the single-pass "onesweep" form: every
// workgroup takes one tile, ranks its keys within the
// tile with wave64 ballots, publishes its per-digit count, resolves the
// counts of all earlier tiles by decoupled look-back, stages the tile in LDS
// in digit order and writes runs of equal digits with consecutive stores.
// The digit histograms of all passes come from one reading pass (fused into
// the key builder in the prepare pipeline).  Tile shapes (threads x keys per
// thread) are template variants; the context picks one (tunable).
#include <algorithm>
#include <map>
#include <mutex>
#include <type_traits>

#include "device_common.h"
#include "internal.h"

namespace snnc {

namespace {

constexpr int RADIX = 256;          // buckets of an 8-bit digit
constexpr int MAX_STRIDE = 512;     // buckets of the widest digit

// look-back status word: [63:62] flag, [61:40] epoch, [39:0] count
constexpr uint64_t FLAG_AGG = 1ull << 62;
constexpr uint64_t FLAG_INC = 2ull << 62;
constexpr uint64_t VALUE_MASK = (1ull << 40) - 1;
constexpr uint32_t EPOCH_MAX = (1u << 22) - 1;

// The lanes of the set v that hold the same digit d: one ballot
// per digit bit (bits above the digit's width are zero in every lane and
// leave the set unchanged).  With the lane's bit as a mask m of all zeros or
// ones, peers & ~(ballot ^ m) is one three-operand bit operation per half.
template <int BITS>
__device__ __forceinline__ uint64_t digit_peers(uint32_t d, uint64_t v) {
    uint32_t lo = (uint32_t)v, hi = (uint32_t)(v >> 32);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)d, b, 1);
        const uint64_t bb = __ballot(m != 0);
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)bb, m, 0x90);          // lo & ~(bb ^ m)
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(bb >> 32), m, 0x90);
    }
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ uint64_t pack_status(uint64_t flag, uint32_t epoch, uint64_t v) {
    return flag | ((uint64_t)epoch << 40) | (v & VALUE_MASK);
}

}  // namespace

namespace {

constexpr int HNT = 1024;

__global__ __launch_bounds__(HNT) void k_hist(const uint64_t* keys, uint64_t n, uint32_t bit_lo, uint32_t bit_hi,
                                              Digits dg, uint64_t* hist) {
    extern __shared__ uint32_t h[];   // a histogram a pass
    for (uint32_t i = threadIdx.x; i < dg.passes * dg.stride; i += HNT) h[i] = 0;
    __syncthreads();
    constexpr int HU = 4;   // independent keys per thread per step: their loads overlap
    for (uint64_t base = (uint64_t)blockIdx.x * HNT * HU; base < n; base += (uint64_t)gridDim.x * HNT * HU) {
        uint64_t k[HU];
#pragma unroll
        for (int u = 0; u < HU; ++u) {
            const uint64_t i = base + (uint64_t)u * HNT + threadIdx.x;
            k[u] = i < n ? keys[i] : 0;
        }
#pragma unroll
        for (int u = 0; u < HU; ++u) {
            const bool valid = base + (uint64_t)u * HNT + threadIdx.x < n;
            for (uint32_t p = 0; p < dg.passes; ++p) {
                const uint32_t s = dg.shift(bit_lo, p);
                const uint32_t mask = (1u << min(bit_hi - s, dg.width(p))) - 1;
                wave_hist_add(&h[p * dg.stride], (uint32_t)((k[u] >> s) & mask), valid);
            }
        }
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < dg.passes * dg.stride; i += HNT)
        if (h[i]) atomicAdd((unsigned long long*)&hist[i], (unsigned long long)h[i]);
}

// exclusive scan over the buckets of each pass (one workgroup per pass)
template <int STRIDE>
__global__ __launch_bounds__(STRIDE) void k_hist_scan(const uint64_t* hist, uint64_t* off) {
    __shared__ uint64_t scratch[STRIDE / 64];
    const uint64_t v = hist[blockIdx.x * STRIDE + threadIdx.x];
    uint64_t tot;
    const uint64_t ex = block_excl_scan<STRIDE, uint64_t>(v, scratch, &tot);
    off[blockIdx.x * STRIDE + threadIdx.x] = ex;
}

// The tile of onesweep workgroup b of `grid`.  Workgroups go to the eight dies
// (each with its own L2) in turn by index; the tiles of every 128 are dealt so
// that a die gets CHUNK = 16 consecutive ones: their runs of equal digits meet
// inside cache lines, and the die's L2 merges both sides of such a line before
// it is written.  The tile is known without a ticket from an atomic counter,
// whose round trip would come before every tile's loads.  Passes over 2^28
// pairs, eight and nine bits: 1346 and 1493 us with 8 tiles to a die, 1334 and
// 1470 with 16, 1493 and 1622 with 32 (tile = index cost a fifth more than 8).
// By the HBM counters a pass moves 24.7 B a pair with eight bits and 25.4 - 25.5 with
// nine, of 24 needed (26.4 - 26.9 and 29.3 with 8192-pair tiles in launch order).
constexpr uint32_t DIES = 8, CHUNK = 16;

// Earlier tiles whose counts a look-back reads at once: a word costs a trip past
// the L2 (the dies share no cache).  2^28 pairs: two 1358 us, four 1346, six 1349.
constexpr int AHEAD = 4;

__device__ __forceinline__ uint32_t pass_tile(uint32_t b, uint32_t grid) {
    const uint32_t first = b / (DIES * CHUNK) * (DIES * CHUNK), r = b - first;
    return first + DIES * CHUNK <= grid ? first + r % DIES * CHUNK + r / DIES : b;
}

// LB = true: onesweep (decoupled look-back, digit_off = exclusive digit totals).
// A workgroup whose look-back meets a tile without counts waits for spin_limit
// polls and then counts its digit in that tile itself, so no order in which
// workgroups start (another kernel may hold a die) can keep it waiting.
// taken_epoch: epoch of the counts it takes (the pass's own; 0, which no pass has,
// where a check wants every earlier tile counted).  LB = false: the scatter of a reduce-then-scan pass
// (tile = block index, digit_off = exclusive scan of the per-tile counts laid
// out digit-major, so entry d * tiles + t is the tile's global base for d).
// RB: buckets of the digit (256, or 512 for 9-bit digits).  SPLIT: stage the
// keys, then the payloads, through one LDS buffer of 8 B per pair that also
// holds the per-wave digit counts while the tile is ranked: about 67 KB for an
// 8192-pair tile (two workgroups a compute unit), 133 KB for 16384 pairs.
// A tile's count is published as soon as it is known and looked back for only
// when the tile stands staged in LDS: by then the earlier tiles have mostly
// published theirs.  Waiting for them before the staging took 40% of a tile's
// time; 2^28 pairs, 8-bit digit, 8192-pair tiles: 1594 us so, 1401 as here
// (16384-pair tiles 1501 and 1334 us: 4.8 TB/s at 24 B per pair, the rate of a
// large copy).
template <int NT, int IPT, bool FINAL, bool LB, int RB, bool SPLIT>
__global__ __launch_bounds__(NT) void k_onesweep(const uint64_t* __restrict__ kin, const uint32_t* __restrict__ vin,
                                                 uint64_t* __restrict__ kout, uint32_t* __restrict__ vout, uint64_t n,
                                                 uint32_t shift, uint32_t dbits, const uint64_t* __restrict__ digit_off,
                                                 uint64_t* lookback, uint32_t epoch, uint32_t taken_epoch,
                                                 uint32_t spin_limit, FinalOut fo) {
    constexpr int TILE = NT * IPT;
    constexpr int WAVES = NT / 64;
    static_assert(NT >= RB, "one thread per digit");
    constexpr int STAGE_K = TILE * 8;            // bytes of the staged keys
    constexpr int WH = WAVES * RB * 4;           // bytes of the per-wave digit counts
    static_assert(!SPLIT || WH <= STAGE_K, "split staging layout");
    __shared__ uint64_t out_base[RB];            // global position of LDS slot 0 if it held digit d (may wrap below 0)
    __shared__ uint64_t scan_scratch[NT / 64];
    __shared__ __align__(16) unsigned char pool[SPLIT ? STAGE_K : STAGE_K + TILE * 4 + WH];
    auto wave_hist = reinterpret_cast<uint32_t (*)[RB]>(SPLIT ? pool : pool + STAGE_K + TILE * 4);
    uint64_t* stage_k = reinterpret_cast<uint64_t*>(pool);
    uint32_t* stage_v = reinterpret_cast<uint32_t*>(SPLIT ? pool : pool + STAGE_K);

    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (uint32_t i = threadIdx.x; i < WAVES * RB; i += NT) (&wave_hist[0][0])[i] = 0;
    __syncthreads();
    const uint64_t tile = LB ? pass_tile(blockIdx.x, gridDim.x) : blockIdx.x;
    const uint64_t base = tile * TILE;
    const uint32_t mask = (1u << dbits) - 1;

    // full: no per-element guards (every tile but the last)
    auto run = [&](auto full_tile) {
        constexpr bool full = decltype(full_tile)::value;
        // striped load within each wave: item k of lane l is element base + wave*64*IPT + k*64 + l
        uint64_t key[IPT];
        uint32_t val[IPT];
        uint32_t rank[IPT];
        const uint64_t wbase = base + (uint64_t)wave * 64 * IPT + lane;
        if constexpr (full) {
#pragma unroll
            for (int k = 0; k < IPT; ++k) key[k] = kin[wbase + (uint64_t)k * 64];
            __builtin_amdgcn_sched_barrier(0);   // keys first: the ranking below waits for them alone
#pragma unroll
            for (int k = 0; k < IPT; ++k) val[k] = vin[wbase + (uint64_t)k * 64];
            __builtin_amdgcn_sched_barrier(0);
        } else {
#pragma unroll
            for (int k = 0; k < IPT; ++k) {
                const uint64_t i = wbase + (uint64_t)k * 64;
                key[k] = i < n ? kin[i] : 0ull;
                val[k] = i < n ? vin[i] : 0u;
            }
        }
        constexpr int MAXBITS = RB == 512 ? 9 : 8;   // digits of a pass have at most this many bits
#pragma unroll
        for (int k = 0; k < IPT; ++k) {
            const bool valid = full || wbase + (uint64_t)k * 64 < n;
            const uint32_t d = (uint32_t)(key[k] >> shift) & mask;
            const uint64_t peers = digit_peers<MAXBITS>(d, full ? ~0ull : __ballot(valid));
            uint32_t r = 0;
            if (valid) {
                const uint32_t before = wave_hist[wave][d];
                r = before + __builtin_amdgcn_mbcnt_hi((uint32_t)(peers >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)peers, 0u));
                // the highest peer advances the wave's counter of this digit
                if ((peers >> lane) == 1ull) wave_hist[wave][d] = r + 1;
            }
            rank[k] = r;
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();

        // per digit: the tile's count, published before anything else, and the slots of its first key and
        // of each wave's first one
        const uint32_t d = threadIdx.x;
        const bool digit_thread = d < RB;
        uint64_t* const my = lookback + tile * RB + d;
        uint32_t cnt = 0;
        if (digit_thread) {
            uint32_t woff[WAVES];
#pragma unroll
            for (int w = 0; w < WAVES; ++w) woff[w] = wave_hist[w][d];
#pragma unroll
            for (int w = 0; w < WAVES; ++w) {
                wave_hist[w][d] = cnt;
                cnt += woff[w];
            }
            if constexpr (LB)
                __hip_atomic_store(my, pack_status(tile ? FLAG_AGG : FLAG_INC, epoch, cnt), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
        }
        uint32_t tot;
        const uint32_t start = block_excl_scan<NT, uint32_t>(cnt, reinterpret_cast<uint32_t*>(scan_scratch), &tot);
        if (digit_thread) out_base[d] = start;
        __syncthreads();
        const uint32_t tile_n = (uint32_t)min((uint64_t)TILE, n - base);
        // slots (with SPLIT the counts share the staging buffer: all slots first)
#pragma unroll
        for (int k = 0; k < IPT; ++k) {
            const uint32_t dk = (uint32_t)(key[k] >> shift) & mask;
            rank[k] += wave_hist[wave][dk] + (uint32_t)out_base[dk];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < IPT; ++k)
            if (full || wbase + (uint64_t)k * 64 < n) {
                stage_k[rank[k]] = key[k];
                if constexpr (!SPLIT) stage_v[rank[k]] = val[k];
            }

        // per digit: look-back over earlier tiles, which had the time of the staging to publish theirs
        if (digit_thread) {
            uint64_t excl = 0;
            if (LB && tile) {
                int64_t pred = (int64_t)tile - 1;
                uint32_t spins = 0;
                bool found = false;
                while (pred >= 0 && !found) {
                    uint64_t st[AHEAD];
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u)
                        st[u] = __hip_atomic_load(lookback + (uint64_t)max(pred - u, (int64_t)0) * RB + d,
                                                  __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const int64_t from = pred;
                    bool ready = true;
#pragma unroll
                    for (int u = 0; u < AHEAD; ++u) {
                        const uint64_t flag = st[u] & (3ull << 62);
                        ready = ready && !found && pred >= 0 && flag != 0 && (uint32_t)((st[u] >> 40) & EPOCH_MAX) == taken_epoch;
                        if (ready) {
                            excl += st[u] & VALUE_MASK;
                            found = flag == FLAG_INC;
                            --pred;
                        }
                    }
                    if (pred != from) continue;
                    if (spins++ >= spin_limit) {   // its keys are all there: every tile before the last is full
                        const uint64_t* pk = kin + (uint64_t)pred * TILE;
                        uint32_t c = 0;
#pragma unroll 1
                        for (int i = 0; i < TILE; ++i) c += ((uint32_t)(pk[i] >> shift) & mask) == d ? 1u : 0u;
                        excl += c;
                        --pred;
                        continue;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
                __hip_atomic_store(my, pack_status(FLAG_INC, epoch, excl + cnt), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            // (LB false: offsets known from the reduce-then-scan counts)
            out_base[d] = (LB ? digit_off[d] + excl : digit_off[(uint64_t)d * ((n + TILE - 1) / TILE) + tile]) - start;
        }
        __syncthreads();
        // every thread writes slots tid, tid + NT, ...: equal digits go to consecutive positions
        uint32_t dd[IPT];   // digits of the thread's slots, kept for the payloads
#pragma unroll
        for (int k = 0; k < IPT; ++k) {
            const uint32_t s = threadIdx.x + (uint32_t)k * NT;
            dd[k] = 0;
            if (full || s < tile_n) {
                const uint64_t x = stage_k[s];
                dd[k] = (uint32_t)(x >> shift) & mask;
                const uint64_t g = out_base[dd[k]] + s;
                if constexpr (FINAL) {
                    if (fo.prefix64) fo.prefix64[g] = x >> fo.tgt_shift;
                    else fo.src[g] = (int32_t)(x >> fo.tgt_shift);
                    fo.tgt[g] = (int32_t)((x >> 16) & fo.tgt_mask);
                    fo.delay[g] = (uint16_t)(x & 0xffffu);
                } else {
                    kout[g] = x;
                }
                if constexpr (!SPLIT) {
                    if constexpr (FINAL) fo.weight[g] = __uint_as_float(stage_v[s]);
                    else vout[g] = stage_v[s];
                }
            }
        }
        if constexpr (SPLIT) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < IPT; ++k)
                if (full || wbase + (uint64_t)k * 64 < n) stage_v[rank[k]] = val[k];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < IPT; ++k) {
                const uint32_t s = threadIdx.x + (uint32_t)k * NT;
                if (full || s < tile_n) {
                    const uint64_t g = out_base[dd[k]] + s;
                    if constexpr (FINAL) fo.weight[g] = __uint_as_float(stage_v[s]);
                    else vout[g] = stage_v[s];
                }
            }
        }
    };
    if (base + TILE <= n) run(std::true_type{});
    else run(std::false_type{});
}

__global__ void k_unpack(const uint64_t* keys, const uint32_t* vals, uint64_t n, FinalOut fo) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint64_t k = keys[i];
    if (fo.prefix64) fo.prefix64[i] = k >> fo.tgt_shift;
    else fo.src[i] = (int32_t)(k >> fo.tgt_shift);
    fo.tgt[i] = (int32_t)((k >> 16) & fo.tgt_mask);
    fo.delay[i] = (uint16_t)(k & 0xffffu);
    fo.weight[i] = __uint_as_float(vals[i]);
}

struct PassArgs {
    const uint64_t* kin;
    const uint32_t* vin;
    uint64_t* kout;
    uint32_t* vout;
    uint64_t n;
    uint32_t shift, dbits;
    const uint64_t* off;
    uint64_t* lookback;
    uint32_t epoch, taken_epoch;
    uint32_t spin_limit;
    FinalOut fo;
    int mode;   // 0: onesweep, 1: reduce-then-scan
};

// Digit counts of every tile of a pass, digit-major (counts[d * tiles + t]),
// for the reduce-then-scan form of a pass.
template <int NT, int IPT, int RB>
__global__ __launch_bounds__(NT) void k_tile_counts(const uint64_t* __restrict__ kin, uint64_t n, uint32_t shift,
                                                    uint32_t dbits, uint32_t* counts) {
    constexpr int TILE = NT * IPT;
    __shared__ uint32_t h[RB];
    for (uint32_t i = threadIdx.x; i < RB; i += NT) h[i] = 0;
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t tiles = (n + TILE - 1) / TILE;
    const uint64_t wbase = (uint64_t)blockIdx.x * TILE + (uint64_t)wave * 64 * IPT + lane;
    const uint32_t mask = (1u << dbits) - 1;
#pragma unroll
    for (int k = 0; k < IPT; ++k) {
        const uint64_t i = wbase + (uint64_t)k * 64;
        const bool valid = i < n;
        const uint32_t d = valid ? (uint32_t)((kin[i] >> shift) & mask) : 0u;
        wave_hist_add(h, d, valid);
    }
    __syncthreads();
    for (uint32_t d = threadIdx.x; d < RB; d += NT) counts[(uint64_t)d * tiles + blockIdx.x] = h[d];
}

template <int NT, int IPT, bool FINAL, bool LB, int RB, bool SPLIT>
void launch_onesweep(Ctx& c, const PassArgs& a, const uint64_t* off) {
    const uint64_t tiles = (a.n + (uint64_t)NT * IPT - 1) / ((uint64_t)NT * IPT);
    hipLaunchKernelGGL((k_onesweep<NT, IPT, FINAL, LB, RB, SPLIT>), dim3((unsigned)tiles), dim3(NT), 0, c.stream, a.kin,
                       a.vin, a.kout, a.vout, a.n, a.shift, a.dbits, off, a.lookback, a.epoch, a.taken_epoch, a.spin_limit, a.fo);
}

template <int NT, int IPT, int RB, bool SPLIT = false>
void launch_pass(Ctx& c, const PassArgs& a, bool final) {
    constexpr int TILE = NT * IPT;
    const uint64_t tiles = (a.n + TILE - 1) / TILE;
    const uint64_t* off = a.off;
    std::vector<void*> temps;
    if (a.mode == 1) {
        // reduce-then-scan: per-tile counts, one scan, scatter with known bases
        uint32_t* counts = dalloc_n<uint32_t>(c, tiles * RB);
        temps.push_back(counts);
        uint64_t* scanned = dalloc_n<uint64_t>(c, tiles * RB + 1);
        temps.push_back(scanned);
        hipLaunchKernelGGL((k_tile_counts<NT, IPT, RB>), dim3((unsigned)tiles), dim3(NT), 0, c.stream, a.kin,
                           a.n, a.shift, a.dbits, counts);
        HIPCHK(hipGetLastError());
        scan_u32_u64(c, counts, scanned, tiles * RB, false);
        off = scanned;
        if (final) launch_onesweep<NT, IPT, true, false, RB, SPLIT>(c, a, off);
        else launch_onesweep<NT, IPT, false, false, RB, SPLIT>(c, a, off);
    } else if (final) {
        launch_onesweep<NT, IPT, true, true, RB, SPLIT>(c, a, off);
    } else {
        launch_onesweep<NT, IPT, false, true, RB, SPLIT>(c, a, off);
    }
    HIPCHK(hipGetLastError());
    for (void* p : temps) dfree(c, p);   // stream-ordered release
}

struct Variant {
    int nt, ipt;
    bool split;   // keys and payloads staged through LDS one after the other
};
// tile shapes available to the tuner; unless one is set, plan_sort takes 8, 0 or
// 12 by the number of pairs: 4096-, 8192- and 16384-pair tiles staged in two phases
constexpr Variant VARIANTS[] = {{512, 16, true},  {256, 8, false},  {512, 8, false}, {512, 16, false},
                                {256, 16, false}, {256, 12, false}, {1024, 8, false}, {1024, 8, true},
                                {512, 8, true},   {512, 12, true},  {256, 16, true},  {512, 11, true},
                                {1024, 16, true}, {768, 12, true}};
constexpr int LARGE_TILE_VARIANT = 12;
constexpr uint64_t LARGE_TILE = (uint64_t)VARIANTS[LARGE_TILE_VARIANT].nt * VARIANTS[LARGE_TILE_VARIANT].ipt;
constexpr int N_VARIANTS = sizeof(VARIANTS) / sizeof(VARIANTS[0]);

// autotuner results for the process: (pass algorithm, tile shape) per size
// class; used by every context whose sort settings were not set by hand
struct TuneKey {
    int size_class;   // floor(log2 n)
    uint32_t bits;
    bool operator<(const TuneKey& o) const { return size_class != o.size_class ? size_class < o.size_class : bits < o.bits; }
};

std::map<TuneKey, std::pair<int, int>>& tune_cache() {
    static std::map<TuneKey, std::pair<int, int>> m;
    return m;
}

int log2_floor(uint64_t n) {
    int l = 0;
    while (n >>= 1) ++l;
    return l;
}

void launch_variant(Ctx& c, int v, const PassArgs& a, bool final, bool wide) {
    if (wide) {   // 9-bit digits: tile shapes with at least 512 threads
        switch (v) {
        case 2: launch_pass<512, 8, 512>(c, a, final); break;
        case 3: launch_pass<512, 16, 512>(c, a, final); break;
        case 0: launch_pass<512, 16, 512, true>(c, a, final); break;
        case 6: launch_pass<1024, 8, 512>(c, a, final); break;
        case 7: launch_pass<1024, 8, 512, true>(c, a, final); break;
        case 8: launch_pass<512, 8, 512, true>(c, a, final); break;
        case 9: launch_pass<512, 12, 512, true>(c, a, final); break;
        case 11: launch_pass<512, 11, 512, true>(c, a, final); break;
        case 12: launch_pass<1024, 16, 512, true>(c, a, final); break;
        case 13: launch_pass<768, 12, 512, true>(c, a, final); break;
        default: raise(SNNC_EINVAL, "9-bit digits need a tile of at least 512 threads");
        }
        return;
    }
    switch (v) {
    case 1: launch_pass<256, 8, RADIX>(c, a, final); break;
    case 2: launch_pass<512, 8, RADIX>(c, a, final); break;
    case 3: launch_pass<512, 16, RADIX>(c, a, final); break;
    case 4: launch_pass<256, 16, RADIX>(c, a, final); break;
    case 5: launch_pass<256, 12, RADIX>(c, a, final); break;
    case 6: launch_pass<1024, 8, RADIX>(c, a, final); break;
    case 7: launch_pass<1024, 8, RADIX, true>(c, a, final); break;
    case 8: launch_pass<512, 8, RADIX, true>(c, a, final); break;
    case 9: launch_pass<512, 12, RADIX, true>(c, a, final); break;
    case 10: launch_pass<256, 16, RADIX, true>(c, a, final); break;
    case 11: launch_pass<512, 11, RADIX, true>(c, a, final); break;
    case 12: launch_pass<1024, 16, RADIX, true>(c, a, final); break;
    case 13: launch_pass<768, 12, RADIX, true>(c, a, final); break;
    default: launch_pass<512, 16, RADIX, true>(c, a, final); break;
    }
}

}  // namespace

// look-back table of the lane: tiles x buckets status words, zeroed once when (re)allocated
void release_lookback(Ctx& c) {
    dfree(c, c.lookback);
    c.lookback = nullptr;
    c.lookback_bytes = 0;
}

void ensure_lookback(Ctx& c, size_t need) {
    if (c.lookback_bytes >= need) return;
    release_lookback(c);
    c.lookback = dalloc(c, need);
    c.lookback_bytes = need;
    HIPCHK(hipMemsetAsync(c.lookback, 0, need, c.stream));
    c.sort_epoch = 0;
}

void next_epoch(Ctx& c) {
    if (++c.sort_epoch > EPOCH_MAX) {
        HIPCHK(hipMemsetAsync(c.lookback, 0, c.lookback_bytes, c.stream));
        c.sort_epoch = 1;
    }
}

int sort_variant_count() { return N_VARIANTS; }

// Pass algorithm, tile shape and digit plan of a sort of n keys over `bits`
// bits: as few passes as the tile shape's digits allow, of equal or nearly equal
// width (a pass costs more the wider its digit).  9-bit digits (512 buckets)
// need a tile of at least 512 threads; 10-bit ones were not worth it (passes over
// 2^28 pairs with the largest tile, when the look-back still came before the staging:
// 8 bits 1501, 9 bits 1642, 10 bits 2070 us; the first two take 1334 and 1470 since).
// The scratch of fixed size (`fixed`) keeps to the tiles its limits are stated for.
SortPlan plan_sort(const Ctx& c, uint64_t n, uint32_t bits, bool fixed) {
    SortPlan p;
    p.variant = (c.sort_variant >= 0 && c.sort_variant < N_VARIANTS) ? c.sort_variant : 0;
    p.mode = c.sort_mode;
    if (!c.sort_pinned) {
        // few tiles: half-size ones, whose ranking is half as long a chain (passes over 1e5, 3e5, 1e6
        // pairs: 12.5, 14.5, 20.7 us against 14.6, 16.8, 21.9 with the full size; 3e6 pairs 29.3 against 27.4)
        if (p.variant == 0 && n < (1u << 20) + (1u << 19)) p.variant = 8;
        // many: double-size ones, whose runs fill whole lines (8 bits, 2^26, 2^27, 2^28 pairs: 339, 674,
        // 1334 us against 335, 678, 1363; 9 bits, 2^23, 2^25, 2^28: 60, 197, 1470 against 55, 213, 1716)
        const bool nine = (bits + 8) / 9 < (bits + 7) / 8;
        if (p.variant == 0 && n >= (nine ? 1ull << 25 : 1ull << 27) && !fixed) p.variant = LARGE_TILE_VARIANT;
        auto it = tune_cache().find(TuneKey{log2_floor(std::max<uint64_t>(n, 1)), bits});
        if (it != tune_cache().end()) {
            p.mode = it->second.first;
            p.variant = it->second.second;
        }
    }
    const uint32_t p8 = (bits + 7) / 8, p9 = (bits + 8) / 9;
    const bool can9 = VARIANTS[p.variant].nt >= 512;
    Digits& d = p.d;
    if (can9 && c.digit_bits == 9) {          // forced: every pass 9 bits
        d.passes = p9;
        d.dbits = 9;
    } else {
        d.passes = c.digit_bits != 8 && can9 ? p9 : p8;
        d.dbits = d.passes ? bits / d.passes : 0;
        d.n_long = d.passes ? bits % d.passes : 0;
    }
    d.stride = std::max<uint32_t>(256, 1u << (d.dbits + (d.n_long ? 1 : 0)));
    return p;
}

// Timer name of a radix-sort step: "sort_<step>", or "<sort_tag>_<step>" for
// the sorts that generation runs (kept out of the Prepare phase's figures).
std::string sort_timer(const Ctx& c, const char* step) {
    return std::string(c.sort_tag ? c.sort_tag : "sort") + "_" + step;
}

// Workgroups of a pass that builds digit histograms of n keys: every workgroup
// ends with one global atomic per non-empty bucket and pass (about 5e10/s over
// the device), so it takes 8192 keys, fewer only below 512 workgroups, and is
// large (512 or 1024 threads) so that these fill the compute units.
// 3e6 keys in 5 digits: 100 us with 4096 workgroups of 256 threads, 40 with 1024, 23
// with 512 of 1024 threads.
uint32_t hist_grid(uint64_t n) {
    const uint64_t per = std::min<uint64_t>(std::max<uint64_t>(n / 512, 1024), 8192);
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((n + per - 1) / per, 8192));
}

void launch_hist(Ctx& c, const uint64_t* keys, uint64_t n, uint32_t bit_lo, uint32_t bit_hi,
                 const Digits& dg, uint64_t* hist) {
    HIPCHK(hipMemsetAsync(hist, 0, (size_t)dg.passes * dg.stride * 8, c.stream));
    const uint32_t grid = hist_grid(n);
    tstart(c, sort_timer(c, "hist").c_str());
    hipLaunchKernelGGL(k_hist, dim3(grid), dim3(HNT), dg.passes * dg.stride * 4, c.stream, keys, n, bit_lo, bit_hi, dg, hist);
    tstop(c);
    HIPCHK(hipGetLastError());
}

namespace {

__global__ void k_fill_words(uint64_t* p, uint64_t n, uint64_t v) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// clears n 64-bit words with a kernel (no memset node in a captured stream)
void fill_words(Ctx& c, uint64_t* p, uint64_t n) {
    if (!n) return;
    const unsigned grid = (unsigned)std::min<uint64_t>((n + 255) / 256, 4096);
    hipLaunchKernelGGL(k_fill_words, dim3(grid), dim3(256), 0, c.stream, p, n, 0ull);
    HIPCHK(hipGetLastError());
}

// passes whose digit differs between keys (the others leave the order unchanged);
// hh: their digit histograms, or null when they were not read back
uint32_t live_passes(const uint64_t* hh, const Digits& dg, uint64_t n, uint32_t* live) {
    uint32_t n_live = 0;
    for (uint32_t p = 0; p < dg.passes; ++p) {
        bool trivial = false;
        for (uint32_t b = 0; hh && b < dg.stride; ++b)
            if (hh[(size_t)p * dg.stride + b] == n) trivial = true;
        if (!trivial) live[n_live++] = p;
    }
    return n_live;
}

// Scratch of a sort that allocates nothing: digit histograms and offsets and
// the look-back table, all at fixed addresses; the look-back epoch persists
// with the table.
struct FixedScratch {
    uint64_t* hist;
    uint64_t* off;
    void* lookback;
    size_t lookback_bytes;
    uint32_t* epoch;
};

int radix_sort_impl(Ctx& c, uint64_t* keys0, uint32_t* vals0, uint64_t* keys1, uint32_t* vals1, uint64_t n,
                    uint32_t bit_lo, uint32_t bit_hi, const uint64_t* digit_hist, const FinalOutFn& final_out,
                    bool wait_for_plan, const FixedScratch* fs) {
    const SortPlan plan = plan_sort(c, n, bit_hi > bit_lo ? bit_hi - bit_lo : 0, fs != nullptr);
    const Digits& dg = plan.d;
    const uint32_t passes = dg.passes;
    // the reduce-then-scan passes allocate per-tile counts: fixed scratch takes onesweep passes
    int variant = plan.variant;
    const int mode = fs ? 0 : plan.mode;
    const uint32_t rb = dg.stride;
    if (passes > 8) raise(SNNC_EUNSUPPORTED, "radix sort over more than 64 bits");
    if (!n) {   // no tile to launch
        c.sort_passes = 0;
        return 0;
    }
    const uint64_t tile = (uint64_t)VARIANTS[variant].nt * VARIANTS[variant].ipt;
    const uint64_t tiles = (n + tile - 1) / tile;
    if (fs && passes && n && (size_t)tiles * rb * 8 > fs->lookback_bytes)
        raise(SNNC_EINVAL, "sort of " + std::to_string(n) + " keys needs a look-back table of " +
                               std::to_string((size_t)tiles * rb * 8) + " bytes, above the " +
                               std::to_string(fs->lookback_bytes) + " of the static scratch");
    void* temps[2] = {nullptr, nullptr};
    auto cleanup = [&] {
        for (void* p : temps) dfree(c, p);
    };
    void* lookback = fs ? fs->lookback : c.lookback;
    uint32_t& epoch = fs ? *fs->epoch : c.sort_epoch;
    const size_t lookback_bytes = fs ? fs->lookback_bytes : 0;
    int cur = 0;
    try {
        uint64_t hh[8 * MAX_STRIDE];
        uint64_t* off = nullptr;
        if (passes) {
            uint64_t* hist = const_cast<uint64_t*>(digit_hist);
            if (!hist && fs) {
                hist = fs->hist;
                fill_words(c, hist, (uint64_t)passes * dg.stride);
                const uint32_t grid = hist_grid(n);
                hipLaunchKernelGGL(k_hist, dim3(grid), dim3(HNT), passes * dg.stride * 4, c.stream, keys0, n, bit_lo,
                                   bit_hi, dg, hist);
                HIPCHK(hipGetLastError());
            } else if (!hist) {
                hist = dalloc_n<uint64_t>(c, (uint64_t)passes * dg.stride);
                temps[0] = hist;
                launch_hist(c, keys0, n, bit_lo, bit_hi, dg, hist);
            }
            if (fs) {
                off = fs->off;
            } else {
                off = dalloc_n<uint64_t>(c, (uint64_t)passes * dg.stride);
                temps[1] = off;
            }
            tstart(c, sort_timer(c, "hist_scan").c_str());
            if (dg.stride == 512)
                hipLaunchKernelGGL(k_hist_scan<512>, dim3(passes), dim3(512), 0, c.stream, hist, off);
            else
                hipLaunchKernelGGL(k_hist_scan<256>, dim3(passes), dim3(256), 0, c.stream, hist, off);
            tstop(c);
            HIPCHK(hipGetLastError());
            if (wait_for_plan) download(c, hh, hist, (size_t)passes * dg.stride * 8);
            if (!fs) {
                try {
                    ensure_lookback(c, (size_t)tiles * rb * 8);
                } catch (const Error&) {
                    // no room for this table (0.5 or 1 B a pair with 4,096-pair tiles): that of the
                    // largest tiles is a quarter of it, and the order is the same
                    const uint64_t large = (n + LARGE_TILE - 1) / LARGE_TILE;
                    if (large >= tiles) throw;
                    ensure_lookback(c, (size_t)large * rb * 8);
                    variant = LARGE_TILE_VARIANT;
                }
                lookback = c.lookback;
            }
        }
        uint32_t live[8];
        const uint32_t n_live = live_passes(wait_for_plan && passes ? hh : nullptr, dg, n, live);
        c.sort_passes = n_live;
        uint64_t* kb[2] = {keys0, keys1};
        uint32_t* vb[2] = {vals0, vals1};
        for (uint32_t li = 0; li < n_live; ++li) {
            const uint32_t p = live[li];
            if (!fs) {
                next_epoch(c);
            } else if (++epoch > EPOCH_MAX) {
                fill_words(c, static_cast<uint64_t*>(lookback), lookback_bytes / 8);
                epoch = 1;
            }
            const bool last = (li + 1 == n_live) && final_out;
            const uint32_t shift = dg.shift(bit_lo, p), width = std::min(bit_hi - shift, dg.width(p));
            PassArgs a{kb[cur], vb[cur], kb[cur ^ 1], vb[cur ^ 1], n, shift, width,
                       off + (size_t)p * dg.stride, (uint64_t*)lookback, epoch, c.lookback_recount ? 0u : epoch,
                       c.lookback_spins, last ? final_out(cur) : FinalOut{}, mode};
            tstart(c, sort_timer(c, last ? "pass_final" : "pass").c_str());
            launch_variant(c, variant, a, last, width > 8);
            tstop(c);
            HIPCHK(hipGetLastError());
            cur ^= 1;
        }
        if (final_out && !n_live) {
            tstart(c, sort_timer(c, "unpack").c_str());
            hipLaunchKernelGGL(k_unpack, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c.stream, kb[cur], vb[cur], n,
                               final_out(cur));
            tstop(c);
            HIPCHK(hipGetLastError());
        }
    } catch (...) {
        cleanup();
        throw;
    }
    cleanup();
    return cur;
}

}  // namespace

int radix_sort(Ctx& c, uint64_t* keys0, uint32_t* vals0, uint64_t* keys1, uint32_t* vals1, uint64_t n,
               uint32_t bit_lo, uint32_t bit_hi, const uint64_t* digit_hist, const FinalOutFn& final_out,
               bool wait_for_plan) {
    return radix_sort_impl(c, keys0, vals0, keys1, vals1, n, bit_lo, bit_hi, digit_hist, final_out, wait_for_plan,
                           nullptr);
}

}  // namespace snnc

// ------------------------------------------------------------------ autotuner
namespace snnc {
namespace {

__global__ void k_random_keys(uint64_t* keys, uint32_t* vals, uint64_t n, uint32_t bit_lo, uint32_t bits,
                              uint32_t seed) {
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint4 b = draw(seed, 0x7ea5u, i, PURPOSE_IDX);
    const uint64_t r = ((uint64_t)b.y << 32) | b.x;
    keys[i] = bits >= 64 ? r : ((r & ((1ull << bits) - 1)) << bit_lo);
    vals[i] = (uint32_t)i;
}

}  // namespace

// Time every (pass algorithm, tile shape) on n synthetic keys with `bits`
// sorted bits; keep the fastest in the context and in the process cache.
void autotune_sort(Ctx& c, uint64_t n, uint32_t bits, int* mode_out, int* variant_out, float* ms_out) {
    const TuneKey key{log2_floor(std::max<uint64_t>(n, 1)), bits};
    auto it = tune_cache().find(key);
    if (it != tune_cache().end()) {
        c.sort_mode = it->second.first;
        c.sort_variant = it->second.second;
        *mode_out = c.sort_mode;
        *variant_out = c.sort_variant;
        *ms_out = -1.f;
        return;
    }
    uint64_t* k0 = dalloc_n<uint64_t>(c, n);
    uint64_t* k1 = dalloc_n<uint64_t>(c, n);
    uint32_t* v0 = dalloc_n<uint32_t>(c, n);
    uint32_t* v1 = dalloc_n<uint32_t>(c, n);
    hipEvent_t a, b;
    HIPCHK(hipEventCreate(&a));
    HIPCHK(hipEventCreate(&b));
    int best_mode = 0, best_var = 0;
    float best = 1e30f;
    const int saved_mode = c.sort_mode, saved_var = c.sort_variant;
    const bool saved_timing = c.timing, saved_pinned = c.sort_pinned;
    c.timing = false;
    c.sort_pinned = true;   // each candidate runs as set
    try {
        for (int mode = 0; mode < 2; ++mode) {
            for (int v = 0; v < N_VARIANTS; ++v) {
                c.sort_mode = mode;
                c.sort_variant = v;
                float t_best = 1e30f;
                for (int rep = 0; rep < 2; ++rep) {
                    hipLaunchKernelGGL(k_random_keys, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c.stream, k0, v0,
                                       n, 16, bits, 1234u);
                    HIPCHK(hipGetLastError());
                    HIPCHK(hipEventRecord(a, c.stream));
                    radix_sort(c, k0, v0, k1, v1, n, 16, 16 + bits, nullptr, nullptr);
                    HIPCHK(hipEventRecord(b, c.stream));
                    HIPCHK(hipEventSynchronize(b));
                    float ms = 0.f;
                    HIPCHK(hipEventElapsedTime(&ms, a, b));
                    t_best = std::min(t_best, ms);
                }
                if (t_best < best) {
                    best = t_best;
                    best_mode = mode;
                    best_var = v;
                }
            }
        }
    } catch (...) {
        c.sort_mode = saved_mode;
        c.sort_variant = saved_var;
        c.timing = saved_timing;
        c.sort_pinned = saved_pinned;
        (void)hipEventDestroy(a);
        (void)hipEventDestroy(b);
        dfree(c, k0); dfree(c, k1); dfree(c, v0); dfree(c, v1);
        throw;
    }
    c.timing = saved_timing;
    c.sort_pinned = saved_pinned;
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    dfree(c, k0); dfree(c, k1); dfree(c, v0); dfree(c, v1);
    c.sort_mode = best_mode;
    c.sort_variant = best_var;
    tune_cache()[key] = {best_mode, best_var};
    *mode_out = best_mode;
    *variant_out = best_var;
    *ms_out = best;
}

}  // namespace snnc

extern "C" snnc_status snnc_autotune_sort(snnc_ctx* ctx, uint64_t n, uint32_t bits, int32_t* mode_out,
                                          int32_t* variant_out, float* ms_out) {
    using namespace snnc;
    if (!ctx || !mode_out || !variant_out || !ms_out || bits == 0 || bits > 48) return SNNC_EINVAL;
    try {
        HIPCHK(hipSetDevice(ctx->device));
        int m = 0, v = 0;
        float ms = 0.f;
        autotune_sort(*ctx, std::max<uint64_t>(n, 1), bits, &m, &v, &ms);
        *mode_out = m;
        *variant_out = v;
        *ms_out = ms;
        return SNNC_OK;
    } catch (const Error& e) {
        ctx->last_error = e.msg;
        return e.code;
    }
}

extern "C" snnc_status snnc_sort_pairs(snnc_ctx* ctx, uint64_t* keys, uint32_t* vals, uint64_t* keys_tmp,
                                       uint32_t* vals_tmp, uint64_t n, uint32_t bit_lo, uint32_t bit_hi,
                                       int32_t* result_in_tmp) {
    using namespace snnc;
    if (!ctx || !result_in_tmp || (n && (!keys || !vals || !keys_tmp || !vals_tmp)) || bit_hi > 64 || bit_lo > bit_hi)
        return SNNC_EINVAL;
    try {
        HIPCHK(hipSetDevice(ctx->device));
        *result_in_tmp = radix_sort(*ctx, keys, vals, keys_tmp, vals_tmp, n, bit_lo, bit_hi, nullptr, nullptr);
        HIPCHK(hipStreamSynchronize(ctx->stream));
        return SNNC_OK;
    } catch (const Error& e) {
        ctx->last_error = e.msg;
        return e.code;
    }
}

// ------------------------------------------------------------------ allocation-free sort
// One static scratch array per GPU, for callers that cannot allocate device
// memory.  Layout: digit histograms (8 passes x 512 u64), their offsets
// (same), then the look-back table.  Host code reaches it only through the address that
// hipGetSymbolAddress gives for the current device.
namespace snnc {
namespace {

constexpr size_t NA_BYTES = 16u << 20;
constexpr size_t NA_HIST = 0;
constexpr size_t NA_OFF = NA_HIST + 8 * MAX_STRIDE * 8;
constexpr size_t NA_LB = NA_OFF + 8 * MAX_STRIDE * 8 + 256;   // (256 B spare)
constexpr size_t NA_LB_BYTES = NA_BYTES - NA_LB;
constexpr int NA_MAX_DEVICES = 64;

struct NoallocDevice {
    char* ptr = nullptr;    // device address of `scratch` on this GPU
    uint32_t epoch = 0;     // look-back epoch of the last pass run on it
};

std::mutex& na_mutex() {
    static std::mutex m;
    return m;
}

NoallocDevice* na_devices() {
    static NoallocDevice d[NA_MAX_DEVICES];
    return d;
}

}  // namespace
}  // namespace snnc

static __device__ __align__(256) unsigned char scratch[snnc::NA_BYTES];

namespace snnc {

// Called by snnc_init with the context's device current: takes the device
// address of the static scratch once per device and clears its look-back
// table (a fill kernel on the context stream, waited for).
void noalloc_setup(Ctx& c) {
    if (c.device < 0 || c.device >= NA_MAX_DEVICES) return;
    std::lock_guard<std::mutex> lock(na_mutex());
    NoallocDevice& d = na_devices()[c.device];
    if (d.ptr) return;
    void* p = nullptr;
    HIPCHK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    char* base = static_cast<char*>(p);
    fill_words(c, reinterpret_cast<uint64_t*>(base + NA_LB), NA_LB_BYTES / 8);
    HIPCHK(hipStreamSynchronize(c.stream));
    d.ptr = base;
    d.epoch = 0;
}

}  // namespace snnc

extern "C" snnc_status snnc_sort_pairs_noalloc(snnc_ctx* ctx, uint64_t* keys, uint32_t* vals, uint64_t* keys_tmp,
                                               uint32_t* vals_tmp, uint64_t n, uint32_t bit_lo, uint32_t bit_hi,
                                               int32_t* result_in_tmp) {
    using namespace snnc;
    if (!ctx || !result_in_tmp || (n && (!keys || !vals || !keys_tmp || !vals_tmp)) || bit_hi > 64 || bit_lo > bit_hi)
        return SNNC_EINVAL;
    try {
        HIPCHK(hipSetDevice(ctx->device));
        if (ctx->device < 0 || ctx->device >= NA_MAX_DEVICES) raise(SNNC_EUNSUPPORTED, "device ordinal above 63");
        std::lock_guard<std::mutex> lock(na_mutex());
        NoallocDevice& d = na_devices()[ctx->device];
        if (!d.ptr) raise(SNNC_ESTATE, "static scratch not set up on this device");
        FixedScratch fs{reinterpret_cast<uint64_t*>(d.ptr + NA_HIST), reinterpret_cast<uint64_t*>(d.ptr + NA_OFF),
                        d.ptr + NA_LB, NA_LB_BYTES, &d.epoch};
        const int saved_timing = ctx->timing;
        ctx->timing = 0;   // timing brackets would create events
        int which = 0;
        try {
            which = radix_sort_impl(*ctx, keys, vals, keys_tmp, vals_tmp, n, bit_lo, bit_hi, nullptr, nullptr, true,
                                    &fs);
        } catch (...) {
            ctx->timing = saved_timing;
            throw;
        }
        ctx->timing = saved_timing;
        HIPCHK(hipStreamSynchronize(ctx->stream));
        *result_in_tmp = which;
        return SNNC_OK;
    } catch (const Error& e) {
        ctx->last_error = e.msg;
        return e.code;
    }
}

// The HBM block cache's slot table resolved on the GPU: the same LRU as the
// host-side ss_cache (Section 3.1 names LRU; the replacement details are
// the ones stated for ss_cache_resolve), with its state in HBM, so a
// decode step needs no host round trip between selection and gather.
//
// One workgroup per (sequence, KV head) unit:
//   1. the selection is checked (ascending, -1 padding, blocks below the
//      sequence's count, no more than the unit's capacity); a malformed one
//      raises the error flag and leaves the unit untouched;
//   2. hits are looked up in the unit's block table and refresh their last
//      use; the hit slots are marked in an LDS bitmap;
//   3. misses, ranked in ascending block order, take the unit's empty slots
//      first (in slot order);
//   4. the remaining r victims are the r smallest keys (last use, slot) among
//      the occupied, unmarked slots.  A binary search over last-use values
//      finds the threshold T with at least r keys at or below it; the victims
//      are all keys below T and the lowest slots at T; each victim's rank
//      among them orders the assignment;
//   5. miss q takes empty slot q, or the victim of rank q - empties; the
//      evicted blocks leave the block table; the unit's miss rows (b, g,
//      block, slot), in ascending block order, go to the unit's own region
//      of the miss buffer, with their count.
//
// What bounds it is latency: a chain of dependent loads (the unit's bounds,
// its selection, the table entries) and the exchanges between its waves.  So
// every load that can be made before its use is certain is made at the start
// (the last uses of all slots come with the table entries), the last uses
// stay in registers, and counts and ranks are ballots within a wave with one
// LDS exchange of the waves' totals and one barrier each: a probe of the
// binary search is PS compares and a barrier.  Victims are ranked on packed
// 32-bit (last use, slot) keys read four at a time; last uses that span 2^19
// steps or more take the two-word comparison.  Miss totals are kept per unit
// (one word that all units added to cost 0.9 us of 12.6).  192 units with
// k = 512 and 1024 slots, half of the selection missed, launches back to
// back: 30.6 us before (last uses in LDS, two barriers and a scan per probe,
// keys looked up through the slot list in the ranking), 11.7 us now.
#include <algorithm>
#include <numeric>
#include <vector>

#include "internal.hpp"

namespace {

constexpr int KMAX = 512;         // selections per unit
constexpr int CMAX = 8192;        // slots per unit
constexpr int SLOT_BITS = 13;     // CMAX = 2^13
constexpr int ERR_SELECTION = 1;  // error flag bits
constexpr int ERR_CAPACITY = 2;

// lanes below this one in `mask`
__device__ __forceinline__ int lanes_below(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0));
}

// NT threads (NT >= k: thread t owns entry t of the selection), PS slots per
// thread in registers (NT * PS >= the largest capacity): wave w owns the
// slots [w*64*PS, (w+1)*64*PS), lane l of it the slots i*64 + l of those, so
// ranks in slot order are ballots within the wave plus the waves' totals.
template <int NT, int PS>
__global__ __launch_bounds__(NT) void resolve_kernel(const int32_t *__restrict__ sel, int k, int32_t step, int u0,
                                                     int Hkv, const int32_t *__restrict__ nblk,
                                                     const int64_t *__restrict__ slot_base,
                                                     const int64_t *__restrict__ block_base,
                                                     const int32_t *__restrict__ cap,
                                                     const int32_t *__restrict__ table_room, int32_t *used,
                                                     int32_t *slot_block, int32_t *slot_last, int32_t *block_slot,
                                                     int32_t *__restrict__ slots_out, int32_t *__restrict__ miss_out,
                                                     int32_t *__restrict__ counts, int32_t *err,
                                                     int64_t *total)
{
    constexpr int NW = NT / 64;
    __shared__ uint32_t s_mark[NT * PS / 32];              // slots hit in this call
    __shared__ __align__(16) uint32_t s_key[NT + 4];       // victims in slot order: (last use - lo, slot)
    __shared__ int32_t s_last[NT];                         // their last uses, where those do not fit the key
    __shared__ int32_t s_sorted[NT];                       // victims by (last use, slot)
    __shared__ int s_check[NW], s_miss[NW], s_count[2][NW], s_below[NW], s_at[NW];
    __shared__ uint32_t s_lo[NW], s_hi[NW];

    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int u = u0 + blockIdx.x;  // absolute unit
    const int b = u / Hkv, g = u - b * Hkv;
    const int32_t *su = sel + (int64_t)blockIdx.x * k;  // rows of this call's units
    const int32_t j = t < k ? su[t] : -1;
    const int32_t before = t > 0 && t < k ? su[t - 1] : -1;
    const int C = min(cap[u], NT * PS);
    const int n = min(nblk[b], table_room[b]);
    const int used_old = min(used[u], C);  // read before any barrier: thread 0 rewrites it at the end
    const int64_t total_old = total[u];
    int32_t *out = slots_out + (int64_t)blockIdx.x * k;
    int32_t *rows = miss_out + (int64_t)u * k * 4;
    int32_t *bs = block_slot + block_base[u];
    int32_t *sb = slot_block + slot_base[u];
    int32_t *sl = slot_last + slot_base[u];

    // last uses of the thread's slots, wanted only if there are evictions:
    // loaded now, they arrive with the selection's table entries
    const int s0 = wave * (64 * PS) + lane;
    uint32_t last[PS];
#pragma unroll
    for (int i = 0; i < PS; ++i) last[i] = s0 + i * 64 < used_old ? (uint32_t)sl[s0 + i * 64] : 0xFFFFFFFFu;
    int32_t hit = j >= 0 && j < n ? bs[j] : -1;

    // 1. check the selection
    for (int i = t; i < NT * PS / 32; i += NT) s_mark[i] = 0u;
    const bool bad_t = j < 0 ? (j != -1) : (j >= n || (t > 0 && (before < 0 || before >= j)));
    const int check = __popcll(__ballot(j >= 0)) | (__ballot(bad_t) ? 1 << 16 : 0);
    if (lane == 0) s_check[wave] = check;
    __syncthreads();
    int valid = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) valid += s_check[w];
    if (valid > C) {  // a malformed selection counts 2^16 per wave that saw it
        if (t < k) out[t] = -1;
        if (t == 0) {
            counts[u] = 0;
            atomicOr(err, (valid >> 16) ? ERR_SELECTION : ERR_CAPACITY);
        }
        return;
    }

    // 2., 3. mark the hits; rank the misses in entry (ascending block) order
    if (hit >= 0) atomicOr(&s_mark[hit >> 5], 1u << (hit & 31));
    const bool is_miss = j >= 0 && hit < 0;
    const unsigned long long miss_mask = __ballot(is_miss);
    if (lane == 0) s_miss[wave] = __popcll(miss_mask);
    __syncthreads();
    int m = 0, q = lanes_below(miss_mask);
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int c = s_miss[w];
        m += c;
        q += w < wave ? c : 0;
    }
    const int empties = min(m, C - used_old);
    const int r = m - empties;  // evictions

    // 4. victims: the r smallest (last use, slot) among occupied, unmarked slots
    if (r > 0) {
        uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
        for (int i = 0; i < PS; ++i) {
            const int s = s0 + i * 64;
            if ((s_mark[s >> 5] >> (s & 31)) & 1u) last[i] = 0xFFFFFFFFu;  // not a candidate, above every last use
            lo = min(lo, last[i]);
            hi = max(hi, last[i] == 0xFFFFFFFFu ? 0u : last[i]);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lo = min(lo, (uint32_t)__shfl_xor((int)lo, o));
            hi = max(hi, (uint32_t)__shfl_xor((int)hi, o));
        }
        if (lane == 0) {
            s_lo[wave] = lo;
            s_hi[wave] = hi;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            lo = min(lo, s_lo[w]);
            hi = max(hi, s_hi[w]);
        }
        // smallest T in [lo, hi] with count(last <= T) >= r.  The counts
        // alternate between two buffers, so one barrier per probe is enough.
        uint32_t T = lo;
        for (int p = 0; T < hi; p ^= 1) {
            const uint32_t mid = T + ((hi - T) >> 1);
            int c = 0;
#pragma unroll
            for (int i = 0; i < PS; ++i) c += __popcll(__ballot(last[i] <= mid));
            if (lane == 0) s_count[p][wave] = c;
            __syncthreads();
            c = 0;
#pragma unroll
            for (int w = 0; w < NW; ++w) c += s_count[p][w];
            if (c >= r) hi = mid;
            else T = mid + 1;
        }
        // all candidates below T, then the lowest slots at T
        int below = 0, at = 0;
#pragma unroll
        for (int i = 0; i < PS; ++i) {
            below += __popcll(__ballot(last[i] < T));
            at += __popcll(__ballot(last[i] == T));
        }
        if (lane == 0) {
            s_below[wave] = below;
            s_at[wave] = at;
        }
        __syncthreads();
        int need = r;  // candidates at T that go
#pragma unroll
        for (int w = 0; w < NW; ++w) need -= s_below[w];
        int pos = 0, at_rank = 0;  // victims, and candidates at T, in the waves before this one
#pragma unroll
        for (int w = 0; w < NW; ++w)
            if (w < wave) {
                pos += s_below[w] + min(s_at[w], max(0, need - at_rank));
                at_rank += s_at[w];
            }
        const bool narrow = T - lo < (1u << (32 - SLOT_BITS));
#pragma unroll
        for (int i = 0; i < PS; ++i) {
            const unsigned long long at_mask = __ballot(last[i] == T);
            const bool take = last[i] < T || (last[i] == T && at_rank + lanes_below(at_mask) < need);
            const unsigned long long take_mask = __ballot(take);
            if (take) {
                const int at_pos = pos + lanes_below(take_mask);
                s_key[at_pos] = narrow ? (last[i] - lo) << SLOT_BITS | (uint32_t)(s0 + i * 64) : (uint32_t)(s0 + i * 64);
                s_last[at_pos] = (int32_t)last[i];
            }
            at_rank += __popcll(at_mask);
            pos += __popcll(take_mask);
        }
        if (t < 4) s_key[r + t] = 0xFFFFFFFFu;  // the rank loop reads four keys at a time
        __syncthreads();
        if (t < r) {
            const uint32_t v = s_key[t];
            int rank = t;  // slot order is the order where all last uses are one
            if (T != lo && narrow) {
                rank = 0;
                for (int w = 0; w < r; w += 4) {
                    const uint4 x = *reinterpret_cast<const uint4 *>(s_key + w);
                    rank += (x.x < v) + (x.y < v) + (x.z < v) + (x.w < v);
                }
            } else if (T != lo) {
                const int32_t lv = s_last[t];
                rank = 0;
                for (int w = 0; w < r; ++w) rank += s_last[w] < lv || (s_last[w] == lv && w < t);
            }
            s_sorted[rank] = (int32_t)(v & (CMAX - 1));
        }
        __syncthreads();
    }

    // 5. assignment and state updates
    if (t < k) {
        int32_t s = hit;
        if (is_miss) {
            if (q < empties) {
                s = used_old + q;
            } else {
                s = s_sorted[q - empties];
                bs[sb[s]] = -1;  // the evicted block leaves the table
            }
            sb[s] = j;
            bs[j] = s;
            int32_t *row = rows + 4 * q;
            row[0] = b;
            row[1] = g;
            row[2] = j;
            row[3] = s;
        }
        if (j >= 0) sl[s] = step;
        out[t] = j >= 0 ? s : -1;
    }
    if (t == 0) {
        used[u] = used_old + empties;
        counts[u] = m;
        total[u] = total_old + m;
    }
}

}  // namespace

struct ss_dev_cache {
    int B = 0, Hkv = 0, units = 0;
    int64_t total_slots = 0, total_table = 0;
    int64_t last_step = INT64_MIN;
    int max_cap = 0;  // largest capacity of any unit
    void *mem = nullptr;  // one device allocation holding every array below
    int64_t *slot_base = nullptr, *block_base = nullptr;
    int64_t *total = nullptr;  // per unit: misses over all resolves
    int32_t *cap = nullptr, *room = nullptr, *used = nullptr, *counts = nullptr, *err = nullptr;
    int32_t *slot_block = nullptr, *slot_last = nullptr, *block_slot = nullptr;
};

namespace {

template <int NT, int PS>
void launch_resolve(ss_dev_cache *c, int64_t step, int u0, int units, const int32_t *sel, int k, const int32_t *nblk,
                    int32_t *slots, int32_t *miss, hipStream_t s)
{
    ss::launch(resolve_kernel<NT, PS>, dim3(units), dim3(NT), s, sel, k, (int32_t)step, u0, c->Hkv, nblk, c->slot_base,
               c->block_base, c->cap, c->room, c->used, c->slot_block, c->slot_last, c->block_slot, slots, miss,
               c->counts, c->err, c->total);
}

// threads for k entries, then slots per thread for the largest region
template <int NT>
void launch_by_capacity(ss_dev_cache *c, int64_t step, int u0, int units, const int32_t *sel, int k,
                        const int32_t *nblk, int32_t *slots, int32_t *miss, hipStream_t s)
{
    const int per = (c->max_cap + NT - 1) / NT;
    if (per <= 2) launch_resolve<NT, 2>(c, step, u0, units, sel, k, nblk, slots, miss, s);
    else if (per <= 4) launch_resolve<NT, 4>(c, step, u0, units, sel, k, nblk, slots, miss, s);
    else if (per <= 8) launch_resolve<NT, 8>(c, step, u0, units, sel, k, nblk, slots, miss, s);
    else launch_resolve<NT, CMAX / NT>(c, step, u0, units, sel, k, nblk, slots, miss, s);
}

}  // namespace

namespace ss {
int32_t *dev_cache_counts(ss_dev_cache *c) { return c->counts; }
int dev_cache_batch(const ss_dev_cache *c) { return c->B; }
int dev_cache_kv_heads(const ss_dev_cache *c) { return c->Hkv; }

ss_status dev_cache_launch(ss_dev_cache *c, int64_t step, int b_begin, int b_end, const int32_t *sel, int k,
                           const int32_t *nblk, int32_t *slots, int32_t *miss, hipStream_t s)
{
    const int units = (b_end - b_begin) * c->Hkv;
    if (units == 0) return SS_OK;
    if (k <= 256) launch_by_capacity<256>(c, step, b_begin * c->Hkv, units, sel, k, nblk, slots, miss, s);
    else launch_by_capacity<KMAX>(c, step, b_begin * c->Hkv, units, sel, k, nblk, slots, miss, s);
    return check_launch("ss_dev_cache_resolve");
}

ss_status dev_cache_check_step(ss_dev_cache *c, int64_t step, int k)
{
    SS_CHECK_ARG(k > 0 && k <= KMAX, "ss_dev_cache_resolve: k=%d (1..%d)", k, KMAX);
    SS_CHECK_ARG(step >= 0 && step <= INT32_MAX, "ss_dev_cache_resolve: step %lld outside [0, 2^31)",
                 (long long)step);
    SS_CHECK_ARG(step >= c->last_step, "ss_dev_cache_resolve: step %lld before %lld", (long long)step,
                 (long long)c->last_step);
    c->last_step = step;
    return SS_OK;
}
}  // namespace ss

extern "C" {

ss_status ss_dev_cache_create(int B, int Hkv, const int32_t *table_room, const int32_t *capacity, void *stream,
                              ss_dev_cache **out)
{
    SS_CHECK_ARG(out, "ss_dev_cache_create: null out");
    *out = nullptr;
    SS_CHECK_ARG(B > 0 && Hkv > 0, "ss_dev_cache_create: bad shape B=%d Hkv=%d", B, Hkv);
    SS_CHECK_ARG(table_room && capacity, "ss_dev_cache_create: null pointer");
    const int units = B * Hkv;
    std::vector<int64_t> sbase(units), bbase(units);
    int64_t slots = 0, table = 0;
    for (int u = 0; u < units; ++u) {
        SS_CHECK_ARG(capacity[u] >= 0, "ss_dev_cache_create: capacity[%d] < 0", u);
        SS_CHECK_SUPPORTED(capacity[u] <= CMAX, "ss_dev_cache_create: capacity[%d]=%d > %d", u, capacity[u], CMAX);
        SS_CHECK_ARG(table_room[u / Hkv] >= 0, "ss_dev_cache_create: table_room[%d] < 0", u / Hkv);
        sbase[u] = slots;
        bbase[u] = table;
        slots += capacity[u];
        table += table_room[u / Hkv];
    }
    auto *c = new (std::nothrow) ss_dev_cache;
    if (!c) return ss::fail(SS_ERR_OOM, "ss_dev_cache_create: out of memory");
    c->B = B;
    c->Hkv = Hkv;
    c->units = units;
    c->total_slots = slots;
    c->total_table = table;
    c->max_cap = *std::max_element(capacity, capacity + units);
    // layout: 3 int64 arrays [units]; int32 arrays cap, used, counts [units], room [B], err [1];
    // slot_block, slot_last [slots]; block_slot [table]
    const size_t bytes = 24 * (size_t)units + 4 * (3 * (size_t)units + B + 1) + 8 * (size_t)slots +
                         4 * (size_t)table + 64;
    hipError_t e = hipMalloc(&c->mem, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        delete c;
        return ss::fail(SS_ERR_OOM, "ss_dev_cache_create: hipMalloc(%zu): %s", bytes, hipGetErrorString(e));
    }
    char *p = static_cast<char *>(c->mem);
    c->total = reinterpret_cast<int64_t *>(p);
    c->slot_base = c->total + units;
    c->block_base = c->slot_base + units;
    c->cap = reinterpret_cast<int32_t *>(c->block_base + units);
    c->used = c->cap + units;
    c->counts = c->used + units;
    c->room = c->counts + units;
    c->err = c->room + B;
    c->slot_block = c->err + 1;
    c->slot_last = c->slot_block + slots;
    c->block_slot = c->slot_last + slots;
    const hipStream_t s = ss::as_stream(stream);
    std::vector<int32_t> zeros(units, 0), room(table_room, table_room + B);
    ss_status st = SS_OK;
    e = hipMemcpyAsync(c->slot_base, sbase.data(), 8 * (size_t)units, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(c->block_base, bbase.data(), 8 * (size_t)units, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(c->cap, capacity, 4 * (size_t)units, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(c->used, zeros.data(), 4 * (size_t)units, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(c->counts, zeros.data(), 4 * (size_t)units, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemcpyAsync(c->room, room.data(), 4 * (size_t)B, hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipMemsetAsync(c->err, 0, 4, s);
    if (e == hipSuccess) e = hipMemsetAsync(c->total, 0, 8 * (size_t)units, s);
    if (e == hipSuccess) e = hipMemsetAsync(c->slot_block, 0xFF, 4 * (size_t)slots, s);  // -1: empty
    if (e == hipSuccess) e = hipMemsetAsync(c->slot_last, 0xFF, 4 * (size_t)slots, s);
    if (e == hipSuccess) e = hipMemsetAsync(c->block_slot, 0xFF, 4 * (size_t)table, s);  // -1: not cached
    if (e == hipSuccess) e = hipStreamSynchronize(s);  // the host vectors above go out of scope
    if (e != hipSuccess) {
        (void)hipGetLastError();
        st = ss::fail(SS_ERR_HIP, "ss_dev_cache_create: initialising the state: %s", hipGetErrorString(e));
        (void)hipFree(c->mem);
        delete c;
        return st;
    }
    *out = c;
    return SS_OK;
}

void ss_dev_cache_destroy(ss_dev_cache *c)
{
    if (!c) return;
    if (c->mem) (void)hipFree(c->mem);
    delete c;
}

ss_status ss_dev_cache_resolve(ss_dev_cache *c, int64_t step, int b_begin, int b_end, const int32_t *sel, int k,
                               const int32_t *nblk, int32_t *slots, int32_t *miss, void *stream)
{
    SS_CHECK_ARG(c, "ss_dev_cache_resolve: null cache");
    SS_CHECK_ARG(0 <= b_begin && b_begin <= b_end && b_end <= c->B, "ss_dev_cache_resolve: range [%d, %d) of %d",
                 b_begin, b_end, c->B);
    if (b_begin == b_end) return SS_OK;
    SS_CHECK_ARG(sel && nblk && slots && miss, "ss_dev_cache_resolve: null pointer");
    ss_status st = ss::dev_cache_check_step(c, step, k);
    if (st) return st;
    return ss::dev_cache_launch(c, step, b_begin, b_end, sel, k, nblk, slots, miss, ss::as_stream(stream));
}

ss_status ss_dev_cache_miss_counts(const ss_dev_cache *c, int32_t *counts_host, int32_t *error_flags)
{
    SS_CHECK_ARG(c && counts_host, "ss_dev_cache_miss_counts: null pointer");
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpy(counts_host, c->counts, 4 * (size_t)c->units, hipMemcpyDeviceToHost);
    if (e == hipSuccess && error_flags) e = hipMemcpy(error_flags, c->err, 4, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return ss::fail(SS_ERR_HIP, "ss_dev_cache_miss_counts: %s", hipGetErrorString(e));
    return SS_OK;
}

ss_status ss_dev_cache_export(const ss_dev_cache *c, int32_t *slot_block, int64_t *slot_last)
{
    SS_CHECK_ARG(c && slot_block && slot_last, "ss_dev_cache_export: null pointer");
    std::vector<int32_t> last(c->total_slots);
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpy(slot_block, c->slot_block, 4 * (size_t)c->total_slots, hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(last.data(), c->slot_last, 4 * (size_t)c->total_slots, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return ss::fail(SS_ERR_HIP, "ss_dev_cache_export: %s", hipGetErrorString(e));
    for (int64_t i = 0; i < c->total_slots; ++i) slot_last[i] = slot_block[i] >= 0 ? last[i] : 0;
    return SS_OK;
}

int64_t ss_dev_cache_total_slots(const ss_dev_cache *c) { return c ? c->total_slots : 0; }

ss_status ss_dev_cache_total_misses(const ss_dev_cache *c, int64_t *total)
{
    SS_CHECK_ARG(c && total, "ss_dev_cache_total_misses: null pointer");
    std::vector<int64_t> per_unit;
    try {
        per_unit.resize(c->units);
    } catch (const std::bad_alloc &) {
        return ss::fail(SS_ERR_OOM, "ss_dev_cache_total_misses: out of memory");
    }
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpy(per_unit.data(), c->total, 8 * per_unit.size(), hipMemcpyDeviceToHost);
    if (e != hipSuccess) return ss::fail(SS_ERR_HIP, "ss_dev_cache_total_misses: %s", hipGetErrorString(e));
    *total = std::accumulate(per_unit.begin(), per_unit.end(), (int64_t)0);
    return SS_OK;
}

}  // extern "C"

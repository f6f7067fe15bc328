// One eviction step of the DeltaS retention policy (Section 3.3, Algorithm 1).
//
// kv_select (one workgroup of 1024 threads) turns the cache metadata into a
// keep list without any host round trip:
//   * sinks = first n_sink slots, window = last n_window slots, the rest are
//     candidates;
//   * the candidates form runs of equal chunk id (the cache is in arrival
//     order), each run shares one score; a run's key is
//     (orderable(score), chunk id), bigger = better, unique per run;
//   * span of a run: floor(N (a - a_min) / (a_max - a_min + 1)); each span
//     keeps min(len, quota - (tokens of better runs in the span)) of every run,
//     newest tokens first (ties within a chunk go to the newer position);
//   * the leftover budget is filled the same way over all spans from the
//     tokens not yet kept;
//   * kept slots -> ascending keep list.
// The runs with their first kept slots are the whole decision: the keep list is
// the sinks, the tail of every run and the window, written run by run.
// One workgroup is a serial chain of memory round trips, block-wide scans and
// vector work, so: slot data is read once, in blocks of 4 consecutive slots per
// thread with one 16-byte load (adjacent lanes read adjacent 16 bytes), five
// blocks of 4 Ki slots per round trip and scan (a budget of 16384 tokens and
// what is above it in one step; more do not fit the registers of 16 waves); a
// wave whose 256 slots are all candidates skips the tests for the edges; and
// each run is compared with the others by as many lanes as there are to spare.
// 16509 slots in 165 runs (indexed) 42 -> 28 us, 8317 in 67 21.4 -> 14.7,
// 17408 in 17 25 -> 15 (before: blocks one by one, chunk ids read a second time for
// the keep list, one lane per run).
// With a slot table (the indexed variant) the K and V rows never move: the
// select kernel itself compacts pos, chunk_id and slot (the physical row of
// each logical token) in place and lists the freed physical rows.
// The kept rows then move down in place: slot d receives row keep[d]
// (keep[d] >= d); the shift keep[d] - d never decreases with d.  kv_slide cuts
// every plane into column strips of at most 128 bytes per row.  One wave walks a
// strip's destinations in ascending order, reading a batch of source rows ahead
// of the one it writes: no row is read by a later destination than its own, so
// within a strip the order alone makes the move safe, and strips share no byte:
// no waits, no flags, every byte read and written once.  Where the strips are
// too few to fill the GPU, the destinations are also cut into segments; the
// rows that a segment reads from behind its own end (at most len - M) are copied
// to a staging area first (kv_stage_tails), before any segment writes.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace ds {

constexpr int SEL_THREADS = 1024;
constexpr int SEL_PER = 4;                          // consecutive slots per thread and block
constexpr int SEL_BLOCK = SEL_THREADS * SEL_PER;
constexpr int SEL_SUB = 5;                          // blocks per step of a pass
constexpr int SEL_STEP = SEL_SUB * SEL_BLOCK;
constexpr long long STAGE_AREA = 256ll << 20;       // at most this much staging area for the segments' tails

// pointer into global memory (lets the compiler emit global rather than flat accesses)
#define GPTR(T) __attribute__((address_space(1))) T *
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct KvArgs {
    int32_t *pos;    // written only by the indexed variant
    int32_t *chunk;
    const float *scores;
    int num_chunks, len, M, n_s, n_w, N;
    int32_t *status;   // [0] outcome (0 ok, 1 invariants broken, 2 keep count wrong), [1] skip the moves,
                       // [3] first moved slot
    int32_t *keep, *run_start, *run_bkt, *run_take, *run_from;
    unsigned long long *run_key;
    int32_t *keep_out;
    int32_t *slot;      // indexed variant: physical row of each logical token (NULL: gather variant)
    int32_t *free_out;  // indexed variant: physical rows of the evicted tokens
    int32_t *outcome_out;  // indexed variant: a copy of status[0] for the caller (or NULL)
    char **plane_tab;  // device copy of the plane pointers, read by the moves
    char *planes[KV_MAX_PLANES];
    int n_planes;
};

__device__ __forceinline__ uint32_t orderable(float f) {
    const uint32_t u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Barrier that orders LDS only: the block reductions below exchange partial
// sums through LDS, and a full __syncthreads would also wait for every global
// store in flight (the keep list written in the same loop).
__device__ __forceinline__ void lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Exclusive prefix sum over the 1024 threads of the block.
// Inclusive prefix sum over the 64 lanes of a wave with DPP moves: row
// shifts by 1, 2, 4, 8 within each row of 16 lanes, then the last lane of a
// row added to the next row(s) by row broadcasts (rows 1 and 3 get lane 15,
// rows 2 and 3 lane 31).  Lanes without a source add 0.
__device__ __forceinline__ int wave_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
    return v;
}

// Exclusive prefix sums over the 1024 threads of the block, of N values per
// thread with all of value 0 before value 1 and so on: a scan inside each wave,
// then wave 0 scans the 16 N wave totals, two per lane.
template <int N>
__device__ __forceinline__ void block_excl_scan(int (&x)[N], int *s_tmp, int &total) {
    constexpr int W = SEL_THREADS / 64;
    static_assert(N * W <= 128, "two wave totals per lane");
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    int incl[N];
#pragma unroll
    for (int i = 0; i < N; ++i) incl[i] = wave_incl_scan(x[i]);
    if (lane == 63) {
#pragma unroll
        for (int i = 0; i < N; ++i) s_tmp[i * W + wid] = incl[i];
    }
    lds_sync();
    if (wid == 0) {
        const int e = 2 * lane;
        const bool in = e < N * W;  // N W is even
        const int t0 = in ? s_tmp[e] : 0, t1 = in ? s_tmp[e + 1] : 0;
        const int it = wave_incl_scan(t0 + t1);
        if (in) {
            s_tmp[e] = it - t0 - t1;
            s_tmp[e + 1] = it - t1;
        }
        if (lane == 63) s_tmp[N * W] = it;
    }
    lds_sync();
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = s_tmp[i * W + wid] + incl[i] - x[i];
    total = s_tmp[N * W];
    lds_sync();
}
__device__ __forceinline__ int block_excl_scan(int x, int *s_tmp, int &total) {
    int v[1] = {x};
    block_excl_scan(v, s_tmp, total);
    return v[0];
}

// Same DPP pattern with max; lanes without a source contribute -1 (x >= -1).
__device__ __forceinline__ int wave_incl_max(int v) {
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x111, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x112, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x114, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x118, 0xf, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x142, 0xa, 0xf, false));
    v = max(v, __builtin_amdgcn_update_dpp(-1, v, 0x143, 0xc, 0xf, false));
    return v;
}

// Maximum of x over the lower threads of the block (-1 for thread 0); x >= -1.
__device__ int block_excl_max(int x, int *s_tmp) {
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int incl = wave_incl_max(x);
    const int excl = __shfl(incl, max(lane - 1, 0), 64);
    if (lane == 63) s_tmp[wid] = incl;
    lds_sync();
    if (wid == 0) {
        const int t = lane < SEL_THREADS / 64 ? s_tmp[lane] : -1;
        const int it = wave_incl_max(t);
        const int et = __shfl(it, max(lane - 1, 0), 64);
        if (lane < SEL_THREADS / 64) s_tmp[lane] = lane > 0 ? et : -1;
    }
    lds_sync();
    const int res = max(s_tmp[wid], lane > 0 ? excl : -1);
    lds_sync();
    return res;
}

__device__ long long block_sum_ll(long long x, long long *s_tmp) {
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    if (lane == 0) s_tmp[wid] = x;
    lds_sync();
    long long r = 0;
#pragma unroll
    for (int i = 0; i < SEL_THREADS / 64; ++i) r += s_tmp[i];
    lds_sync();
    return r;
}

// SEL_PER consecutive int32 from [lo, lo + SEL_PER); entries at or past len read as 0.
__device__ __forceinline__ void load_block(const int32_t *p, int lo, int len, int (&out)[SEL_PER]) {
    if (lo + SEL_PER <= len) {
#pragma unroll
        for (int q = 0; q < SEL_PER / 4; ++q) {
            const int4 v = *(const int4 *)(p + lo + 4 * q);
            out[4 * q] = v.x;
            out[4 * q + 1] = v.y;
            out[4 * q + 2] = v.z;
            out[4 * q + 3] = v.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < SEL_PER; ++k) out[k] = (lo + k < len) ? p[lo + k] : 0;
    }
}

struct RunRec {
    unsigned long long key;  // (orderable score, chunk id): bigger is better
    int len;                 // candidate slots of the run
    int bkt;                 // span of the run
};
constexpr int RUN_CAP = 2048;  // runs ranked from LDS
constexpr int SORT_MIN = 512;  // more runs than this (up to RUN_CAP) are ranked by sorting

__global__ __launch_bounds__(SEL_THREADS) void kv_select_kernel(KvArgs a) {
    __shared__ RunRec s_run[RUN_CAP];
    __shared__ int s_start[RUN_CAP], s_take[RUN_CAP], s_from[RUN_CAP], s_ord[RUN_CAP];
    __shared__ int s_keep[SEL_STEP];  // a copy of the keep list's first entries for the indexed variant's move
    __shared__ int s_scan[SEL_SUB * (SEL_THREADS / 64) + 1];
    __shared__ long long s_ll[SEL_THREADS / 64];
    __shared__ int s_bad[SEL_THREADS / 64];  // per wave, written by it alone
    const int tid = threadIdx.x, wid = __builtin_amdgcn_readfirstlane(tid >> 6);

    if (tid == 0) {
        a.status[0] = 0;
        a.status[1] = 0;
        a.status[2] = 0;
    }
    if (tid < a.n_planes) a.plane_tab[tid] = a.planes[tid];

    const int c0 = a.n_s, c1 = a.len - a.n_w;

    // ---- pass 1: cache invariants and runs of equal chunk id among the
    // candidates [c0, c1)
    int R = 0, bad = 0;
    for (int base = 0; base < a.len; base += SEL_STEP) {
        int ch[SEL_SUB][SEL_PER], ps[SEL_SUB][SEL_PER], pc0[SEL_SUB], pp0[SEL_SUB], off[SEL_SUB];
#pragma unroll
        for (int u = 0; u < SEL_SUB; ++u) {
            const int lo = base + u * SEL_BLOCK + tid * SEL_PER;
            load_block(a.chunk, lo, a.len, ch[u]);
            load_block(a.pos, lo, a.len, ps[u]);
            const bool has_prev = lo > 0 && lo <= a.len;
            pc0[u] = has_prev ? a.chunk[lo - 1] : -1;
            pp0[u] = has_prev ? a.pos[lo - 1] : 0;
        }
        unsigned starts[SEL_SUB];  // the slots of the thread's four at which a run starts
#pragma unroll
        for (int u = 0; u < SEL_SUB; ++u) {
            const int lo = base + u * SEL_BLOCK + tid * SEL_PER, wlo = base + u * SEL_BLOCK + wid * 64 * SEL_PER;
            int pc = pc0[u], pp = pp0[u];
            starts[u] = 0;
            if (wlo > c0 && wlo + 64 * SEL_PER <= c1) {  // every slot of the wave is a candidate, and not the first
#pragma unroll
                for (int k = 0; k < SEL_PER; ++k) {
                    bad |= ((unsigned)ch[u][k] >= (unsigned)a.num_chunks) | (ch[u][k] < pc) | (ps[u][k] <= pp);
                    starts[u] |= (unsigned)(ch[u][k] != pc) << k;
                    pc = ch[u][k];
                    pp = ps[u][k];
                }
            } else if (wlo < a.len) {
#pragma unroll
                for (int k = 0; k < SEL_PER; ++k) {
                    const int i = lo + k;
                    if (i < a.len) {
                        if (ch[u][k] < 0 || ch[u][k] >= a.num_chunks) bad = 1;
                        if (i > 0 && (ch[u][k] < pc || ps[u][k] <= pp)) bad = 1;
                        if (i >= c0 && i < c1 && (i == c0 || ch[u][k] != pc)) starts[u] |= 1u << k;
                        pc = ch[u][k];
                        pp = ps[u][k];
                    }
                }
            }
            off[u] = __popc(starts[u]);
        }
        int tot = 0;
        block_excl_scan(off, s_scan, tot);
#pragma unroll
        for (int u = 0; u < SEL_SUB; ++u) {
            int r = R + off[u];
#pragma unroll
            for (int k = 0; k < SEL_PER; ++k) {
                if (starts[u] & (1u << k)) {
                    const int i = base + u * SEL_BLOCK + tid * SEL_PER + k;
                    if (r < RUN_CAP) {  // the run's first slot and chunk, for the keys
                        s_start[r] = i;
                        s_ord[r] = ch[u][k];
                    }
                    a.run_start[r++] = i;
                }
            }
        }
        R += tot;
    }
    const bool wave_bad = __ballot(bad) != 0;
    if ((tid & 63) == 0) s_bad[wid] = wave_bad;
    __syncthreads();
    int any_bad = 0;
#pragma unroll
    for (int w = 0; w < SEL_THREADS / 64; ++w) any_bad |= s_bad[w];
    if (any_bad) {
        if (tid == 0) {
            a.status[0] = 1;
            a.status[1] = 1;
            if (a.outcome_out) *a.outcome_out = 1;
        }
        return;
    }
    if (tid == 0) a.run_start[R] = c1;
    __syncthreads();

    // ---- run keys and spans.  The two ranking passes below compare every run
    // with every other; up to RUN_CAP runs they read a copy of the run table
    // in LDS (one 16-byte read per comparison), beyond that the global one.
    const int ncand = c1 - c0;
    const int a_min = (ncand > 0) ? a.chunk[c0] : 0;
    const int a_max = (ncand > 0) ? a.chunk[c1 - 1] : 0;
    const long long span = (long long)a_max - a_min + 1;
    const int N = max(1, a.N);
    const bool in_lds = R <= RUN_CAP;
    for (int r = tid; r < R; r += SEL_THREADS) {
        const int rs = in_lds ? s_start[r] : a.run_start[r];
        const int re = in_lds ? (r + 1 < R ? s_start[r + 1] : c1) : a.run_start[r + 1];
        const int chn = in_lds ? s_ord[r] : a.chunk[rs];
        const unsigned long long key = ((unsigned long long)orderable(a.scores[chn]) << 32) | (unsigned)chn;
        const int bkt = (int)(((long long)N * (chn - a_min)) / span);
        a.run_key[r] = key;
        a.run_bkt[r] = bkt;
        if (in_lds) s_run[r] = RunRec{key, re - rs, bkt};
    }
    __syncthreads();

    // ---- ranking.  Every run is compared with every other (from the LDS
    // copy up to RUN_CAP runs, else in global memory), except from SORT_MIN to
    // RUN_CAP runs: there the run indices are sorted in LDS (bitonic network;
    // keys are unique, one run per chunk id) and what a run keeps follows from
    // prefix sums over the runs ranked above it.  (Per pass on MI355X: 1024
    // runs compared pairwise take ~230k clocks, sorted ~70k; 17 runs
    // pairwise a few hundred.)
    const bool by_sort = in_lds && R > SORT_MIN;
    int Rp = 1;
    while (Rp < R) Rp <<= 1;
    auto sort_runs = [&](auto before) __attribute__((always_inline)) {
        for (int i = tid; i < Rp; i += SEL_THREADS) s_ord[i] = i;
        lds_sync();
        for (int k = 2; k <= Rp; k <<= 1)
            for (int j = k >> 1; j > 0; j >>= 1) {
                for (int q = tid; q < Rp / 2; q += SEL_THREADS) {
                    const int i = ((q & ~(j - 1)) << 1) | (q & (j - 1)), l = i + j;
                    const int x = s_ord[i], y = s_ord[l];
                    if ((i & k) == 0 ? before(y, x) : before(x, y)) {
                        s_ord[i] = y;
                        s_ord[l] = x;
                    }
                }
                lds_sync();
            }
    };
    // up to SORT_MIN runs: lanes per run in the pairwise comparisons (a power of
    // two, at most a wave), run and place among them of this lane
    int G = 1;
    while (G < 64 && 2 * G * R <= SEL_THREADS) G <<= 1;
    const int gr = tid / G, gi = tid % G;
    auto group_sum = [&](int x) {
        for (int off = 1; off < G; off <<= 1) x += __shfl_xor(x, off, 64);
        return x;
    };
    // sorted positions 2 tid and 2 tid + 1 (Rp <= 2 SEL_THREADS); -1 past R
    const int i0 = 2 * tid, i1 = i0 + 1;
    int tot = 0;

    // ---- per-span quota: a run keeps what the better runs of its span left
    const long long quota = (a.M - a.n_s - a.n_w) / N;
    long long taken = 0;
    if (by_sort) {
        sort_runs([&](int x, int y) {  // x ranks before y: span ascending, key descending
            if (x >= R) return false;
            if (y >= R) return true;
            const RunRec rx = s_run[x], ry = s_run[y];
            return rx.bkt < ry.bkt || (rx.bkt == ry.bkt && rx.key > ry.key);
        });
        const int r0 = i0 < R ? s_ord[i0] : -1, r1 = i1 < R ? s_ord[i1] : -1;
        const int l0 = r0 >= 0 ? s_run[r0].len : 0, l1 = r1 >= 0 ? s_run[r1].len : 0;
        const int b0 = r0 >= 0 ? s_run[r0].bkt : -1, b1 = r1 >= 0 ? s_run[r1].bkt : -1;
        const int bp = (i0 > 0 && i0 <= R) ? s_run[s_ord[i0 - 1]].bkt : -2;
        // slots of the runs ranked before, and where the run's span starts
        const int e0 = block_excl_scan(l0 + l1, s_scan, tot), e1 = e0 + l0;
        const int h0 = (r0 >= 0 && b0 != bp) ? e0 : -1, h1 = (r1 >= 0 && b1 != b0) ? e1 : -1;
        const int hp0 = max(block_excl_max(max(h0, h1), s_scan), h0), hp1 = max(hp0, h1);
        if (r0 >= 0) {
            const int t = (int)min((long long)l0, max(0LL, quota - (e0 - hp0)));
            s_take[r0] = t;
            a.run_take[r0] = t;
            taken += t;
        }
        if (r1 >= 0) {
            const int t = (int)min((long long)l1, max(0LL, quota - (e1 - hp1)));
            s_take[r1] = t;
            a.run_take[r1] = t;
            taken += t;
        }
    } else if (in_lds) {
        int above = 0;
        const RunRec me = s_run[max(0, min(gr, R - 1))];
        // eight records read before they are compared: one LDS round trip per
        // eight runs rather than per run
        for (int r2 = gi; r2 < R; r2 += 8 * G) {
            RunRec o[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) o[q] = s_run[min(r2 + q * G, R - 1)];
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (r2 + q * G < R && o[q].bkt == me.bkt && o[q].key > me.key) above += o[q].len;
        }
        above = group_sum(above);
        if (gr < R && gi == 0) {
            const int t = (int)min((long long)me.len, max(0LL, quota - above));
            a.run_take[gr] = t;
            s_take[gr] = t;
            taken = t;
        }
    } else {
        for (int r = tid; r < R; r += SEL_THREADS) {
            const unsigned long long key = a.run_key[r];
            const int bk = a.run_bkt[r];
            const long long ln = a.run_start[r + 1] - a.run_start[r];
            long long above = 0;
            for (int r2 = 0; r2 < R; ++r2)
                if (a.run_bkt[r2] == bk && a.run_key[r2] > key) above += a.run_start[r2 + 1] - a.run_start[r2];
            const long long t = min(ln, max(0LL, quota - above));
            a.run_take[r] = (int)t;
            taken += t;
        }
    }
    taken = block_sum_ll(taken, s_ll);
    const long long fill = (long long)(a.M - a.n_s - a.n_w) - taken;
    // beyond RUN_CAP runs the fill pass below reads run_take of runs that other
    // waves stored to global memory: a full barrier (workgroup-scope release and
    // acquire of global memory) orders those stores before the reads; the
    // barriers inside block_sum_ll fence LDS only
    __syncthreads();

    // ---- fill with the best remaining tokens over all spans; a run keeps
    // its newest tokens, slots [run_from, run end)
    if (by_sort) {
        sort_runs([&](int x, int y) {  // key descending
            if (x >= R) return false;
            if (y >= R) return true;
            return s_run[x].key > s_run[y].key;
        });
        const int r0 = i0 < R ? s_ord[i0] : -1, r1 = i1 < R ? s_ord[i1] : -1;
        const int t0 = r0 >= 0 ? s_take[r0] : 0, t1 = r1 >= 0 ? s_take[r1] : 0;
        const int m0 = r0 >= 0 ? s_run[r0].len - t0 : 0, m1 = r1 >= 0 ? s_run[r1].len - t1 : 0;
        const int f0 = block_excl_scan(m0 + m1, s_scan, tot), f1 = f0 + m0;  // left in better runs
        if (r0 >= 0) {
            const int from = s_start[r0] + s_run[r0].len - (t0 + (int)min((long long)m0, max(0LL, fill - f0)));
            a.run_from[r0] = from;
            s_from[r0] = from;
        }
        if (r1 >= 0) {
            const int from = s_start[r1] + s_run[r1].len - (t1 + (int)min((long long)m1, max(0LL, fill - f1)));
            a.run_from[r1] = from;
            s_from[r1] = from;
        }
    } else if (in_lds) {
        int above = 0;
        const RunRec me = s_run[max(0, min(gr, R - 1))];
        for (int r2 = gi; r2 < R; r2 += 8 * G) {
            RunRec o[8];
            int tq[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                o[q] = s_run[min(r2 + q * G, R - 1)];
                tq[q] = s_take[min(r2 + q * G, R - 1)];
            }
#pragma unroll
            for (int q = 0; q < 8; ++q)
                if (r2 + q * G < R && o[q].key > me.key) above += o[q].len - tq[q];
        }
        above = group_sum(above);
        if (gr < R && gi == 0) {
            const int tk = s_take[gr];
            const int from = s_start[gr] + me.len - (tk + (int)min((long long)(me.len - tk), max(0LL, fill - above)));
            a.run_from[gr] = from;
            s_from[gr] = from;
        }
    } else {
        for (int r = tid; r < R; r += SEL_THREADS) {
            const unsigned long long key = a.run_key[r];
            const long long ln = a.run_start[r + 1] - a.run_start[r], tk = a.run_take[r];
            long long above = 0;
            for (int r2 = 0; r2 < R; ++r2)
                if (a.run_key[r2] > key) above += (a.run_start[r2 + 1] - a.run_start[r2]) - a.run_take[r2];
            a.run_from[r] = a.run_start[r + 1] - (int)(tk + min(ln - tk, max(0LL, fill - above)));
        }
    }
    __syncthreads();
    auto run_start = [&](int r) { return in_lds ? (r < R ? s_start[r] : c1) : a.run_start[r]; };
    auto run_from = [&](int r) { return in_lds ? s_from[r] : a.run_from[r]; };

    // ---- keep list (ascending) and, indexed, the freed slots: the sinks, of
    // every run the slots from run_from on (those before it are evicted), the
    // window.  A wave writes a run, several waves one where the runs are few, and as
    // many lanes as an average run is long where they are short: a turn of a wave
    // takes 0.35 us however little it writes (8317 slots in 1040 runs 81 -> 62 us with
    // 8 lanes a run, 2080 of 4 tokens 132 -> 90); runs much longer than that are
    // left to whole waves.
    int total_kept = c0;
    int first_move = a.M;  // smallest destination d with keep[d] != d
    const int n_evict = a.len - a.M;
    auto put = [&](int d, int i) __attribute__((always_inline)) {
        if (d >= a.M) return;
        a.keep[d] = i;
        if (a.keep_out) a.keep_out[d] = i;
        if (d < SEL_STEP) s_keep[d] = i;
    };
    for (int i = tid; i < c0; i += SEL_THREADS) put(i, i);
    int gl = 64;  // lanes per run
    while (gl > 4 && (long long)(gl / 2) * R >= ncand) gl >>= 1;
    __shared__ int s_long;  // the batch's long runs, listed in the second half of s_ord
    for (int rb = 0; rb < R; rb += SEL_THREADS) {
        const int r = rb + tid, n = min(R - rb, SEL_THREADS);
        const int from = r < R ? run_from(r) : 0, kept = r < R ? run_start(r + 1) - from : 0;
        int tot = 0;
        const int dst = total_kept + block_excl_scan(kept, s_scan, tot);
        if (kept > 0 && from != dst) first_move = min(first_move, dst);
        s_ord[tid] = dst;
        if (tid == 0) s_long = 0;
        lds_sync();
        constexpr int W = SEL_THREADS / 64;
        const int lane = tid & 63;
        auto put_run = [&](int q, int i0, int step) __attribute__((always_inline)) {
            const int to = s_ord[q], st = run_start(rb + q), fr = run_from(rb + q), en = run_start(rb + q + 1);
            for (int i = fr + i0; i < en; i += step) put(to + i - fr, i);
            if (a.slot) {  // st - to tokens were evicted before this run
                for (int i = st + i0; i < fr; i += step)
                    if (i - to < n_evict) a.free_out[i - to] = a.slot[i];
            }
        };
        if (gl == 64) {
            const int per = max(1, W / n);
            for (int q = wid / per; q < n; q += W / per) put_run(q, wid % per * 64 + lane, 64 * per);
        } else {
            auto is_long = [&](int q) { return run_start(rb + q + 1) - run_start(rb + q) > 8 * gl; };
            if (r < R && is_long(tid)) s_ord[SEL_THREADS + atomicAdd(&s_long, 1)] = tid;
            for (int q = tid / gl; q < n; q += SEL_THREADS / gl)
                if (!is_long(q)) put_run(q, tid % gl, gl);
            lds_sync();
            for (int l = wid; l < s_long; l += W) put_run(s_ord[SEL_THREADS + l], lane, 64);
        }
        lds_sync();
        total_kept += tot;
    }
    for (int i = tid; i < a.n_w; i += SEL_THREADS) put(total_kept + i, c1 + i);
    if (a.n_w > 0 && c1 != total_kept) first_move = min(first_move, total_kept);
    total_kept += a.n_w;
    // ---- moving destinations form the suffix [first_move, M) (keep[d] - d is
    // nondecreasing)
    {
        // minimum over the block: within each wave by lane exchanges, then over
        // the 16 wave results (one LDS atomic per thread would serialize)
        __shared__ int s_first[SEL_THREADS / 64];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) first_move = min(first_move, __shfl_xor(first_move, off, 64));
        if ((tid & 63) == 0) s_first[tid >> 6] = first_move;
        lds_sync();
#pragma unroll
        for (int w = 0; w < SEL_THREADS / 64; ++w) first_move = min(first_move, s_first[w]);
    }
    if (tid == 0) {
        a.status[3] = first_move;
        const bool count_ok = total_kept == a.M;
        if (!count_ok) {  // cannot happen for valid arguments; never move data then
            a.status[0] = 2;
            a.status[1] = 1;
        }
        if (a.outcome_out) *a.outcome_out = count_ok ? 0 : 2;
    }
    // ---- indexed variant: pos, chunk_id and slot move down in place,
    // new[d] = old[keep[d]] for the moving destinations [first_move, M).
    // keep[d] >= d, so a block of destinations only reads at or above its own
    // start; each block reads everything before any thread writes, and the
    // next block's reads lie above what this block writes.
    if (a.slot && total_kept == a.M) {
        __syncthreads();  // the keep list written above by every thread is read below
        const bool one = a.M <= SEL_STEP;  // the whole keep list is in LDS
        constexpr int PER = SEL_STEP / SEL_THREADS;
        for (int base = first_move; base < a.M; base += SEL_STEP) {
            int vp[PER], vc[PER], vs[PER];
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int d = base + k * SEL_THREADS + tid;
                if (d < a.M) {
                    const int src = one ? s_keep[d] : a.keep[d];
                    vp[k] = a.pos[src];
                    vc[k] = a.chunk[src];
                    vs[k] = a.slot[src];
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int d = base + k * SEL_THREADS + tid;
                if (d < a.M) {
                    a.pos[d] = vp[k];
                    a.chunk[d] = vc[k];
                    a.slot[d] = vs[k];
                }
            }
        }
    }
}

struct SlideArgs {
    char *const *plane_tab;
    uint32_t row_bytes, row_units;  // bytes and 16-byte units of one plane row
    int n_planes, strips;           // strips per plane
    int M, n_evict, segments;
    int seg_tail;                   // staged rows kept per segment, at most
    int32_t *pos, *chunk;
    const int32_t *keep, *status;
    char *area;  // [segments - 1][seg_tail][n_planes][row_bytes]
};

// First destination of segment s (the moving destinations [first, M) in equal parts).
__device__ __forceinline__ int seg_begin(const SlideArgs &a, int first, int s) {
    return first + (int)((long long)(a.M - first) * s / a.segments);
}

// The first destination in [0, M] whose source is slot x or later, by the 64
// lanes of a wave together (three rounds for 256 Ki slots).
__device__ __forceinline__ int first_from(const int32_t *keep, int M, int x, int lane) {
    int lo = 0, hi = M;
    while (lo < hi) {
        const int step = (hi - lo + 63) / 64, i = lo + lane * step;
        const int c = __popcll(__ballot(i < hi && keep[i] < x));  // lanes 0 .. c - 1 lie below
        if (c == 0) break;
        const int l = lo;
        lo = l + (c - 1) * step + 1;
        hi = min(hi, l + c * step);
    }
    return lo;
}

// The rows that segment blockIdx.y reads from behind its end, destination e0 +
// blockIdx.x (of at most seg_tail), to the staging area.
__global__ __launch_bounds__(256) void kv_stage_tails_kernel(SlideArgs a) {
    if (a.status[1]) return;
    const int tid = threadIdx.x, s = blockIdx.y, first = a.status[3];
    const int lo = seg_begin(a, first, s), hi = seg_begin(a, first, s + 1);
    const int e0 = max(first_from(a.keep, a.M, hi, tid & 63), lo);
    const int r = blockIdx.x, d = e0 + r;
    if (d >= hi) return;
    const size_t src = (size_t)a.keep[d] * a.row_bytes;
    GPTR(u32x4) dst = (GPTR(u32x4))(a.area + ((size_t)s * a.seg_tail + r) * a.n_planes * a.row_bytes);
    const uint32_t total = a.n_planes * a.row_units;
    for (uint32_t u0 = tid; u0 < total; u0 += 256 * 4) {
        u32x4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t u = min(u0 + 256 * k, total - 1), p = u / a.row_units;
            v[k] = *(GPTR(const u32x4))(a.plane_tab[p] + src + 16u * (u - p * a.row_units));
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (u0 + 256 * k < total) dst[u0 + 256 * k] = v[k];
    }
}

// Wave (segment, plane, strip): destinations of the segment in batches of
// SLIDE_U loads per lane, 64 / LPR rows each; the next batch's rows are on
// their way while the current one is written.  Workgroup 0 moves pos and chunk.
//
// Bound by HBM: 2 bytes of traffic per moved byte, against 4 through the
// staging area that this replaces for small shifts, and no launches that end at
// once, tickets or waits.  Whole evictions (ranking included), before -> now:
// 16384 of 17408 tokens of 64 KiB, 14.5 k of them moved, 393 -> 390 us (5.2 TB/s);
// one chunk of 125 by the paper's policy from 16384 tokens of 64 KiB 758 -> 382,
// from 8192 of 64 KiB 436 -> 227, of 32 KiB 214 -> 81; from 16384 of 8 KiB
// 195 -> 82; 8192 of 8704 tokens of 16 KiB 171 -> 73; half of 32768 tokens of
// 64 KiB 455 -> 444.
// A strip is 128 bytes, one cache line written by one instruction: 64-byte strips
// (twice the waves) took 545 us on the first of these, 256-byte strips 484.
// 12 loads in flight per lane: 8 took 432, 16 410, 32 408; 4 waves per
// workgroup: 2 took 414, 8 734.
constexpr int SLIDE_WAVES = 4;
constexpr int SLIDE_U = 12;

template <int LPR, bool NT>
__global__ __launch_bounds__(64 * SLIDE_WAVES) void kv_slide_kernel(SlideArgs a) {
    constexpr int R = 64 / LPR, N = R * SLIDE_U;  // rows per load, rows per batch
    if (a.status[1]) return;
    const int tid = threadIdx.x, lane = tid & 63, first = a.status[3];
    if (blockIdx.x == 0) {
        // positions and chunk ids, in blocks of destinations: everything read before
        // anything is written, and later blocks only read behind what this one writes
        constexpr int T = 64 * SLIDE_WAVES, PER = 16;
        for (int b = first; b < a.M; b += T * PER) {
            int vp[PER], vc[PER];
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int src = a.keep[min(b + T * k + tid, a.M - 1)];
                vp[k] = a.pos[src];
                vc[k] = a.chunk[src];
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < PER; ++k) {
                const int d = b + T * k + tid;
                if (d < a.M) {
                    a.pos[d] = vp[k];
                    a.chunk[d] = vc[k];
                }
            }
            __syncthreads();
        }
        return;
    }
    const int w = __builtin_amdgcn_readfirstlane((int)(blockIdx.x - 1) * SLIDE_WAVES + (tid >> 6));
    const int per_seg = a.n_planes * a.strips, s = w / per_seg;
    if (s >= a.segments) return;
    const int p = (w - s * per_seg) / a.strips, strip = w - s * per_seg - p * a.strips;
    const int lo = seg_begin(a, first, s), hi = seg_begin(a, first, s + 1);
    if (lo >= hi) return;
    // destinations from e0 on read the staged copy of their row
    const int e0 = s + 1 < a.segments ? max(first_from(a.keep, a.M, hi, lane), lo) : hi;
    const uint32_t unit = (uint32_t)(strip * LPR + lane % LPR);
    const bool mine = unit < a.row_units;  // the last strip of a row may be narrower
    const int lr = lane / LPR;
    GPTR(char) plane = (GPTR(char))a.plane_tab[p] + 16u * min(unit, a.row_units - 1);
    GPTR(const char) staged = (GPTR(const char))a.area + 16u * min(unit, a.row_units - 1) +
                              ((size_t)s * a.seg_tail * a.n_planes + p) * a.row_bytes;
    const size_t staged_row = (size_t)a.n_planes * a.row_bytes;
    auto load_idx = [&](int b, int(&ix)[SLIDE_U]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < SLIDE_U; ++u) ix[u] = ((GPTR(const int32_t))a.keep)[min(b + u * R + lr, hi - 1)];
    };
    auto load = [&](int b, const int(&ix)[SLIDE_U], u32x4(&buf)[SLIDE_U]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < SLIDE_U; ++u) {
            const int d = min(b + u * R + lr, hi - 1);
            GPTR(const char) src = d < e0 ? (GPTR(const char))plane + (size_t)ix[u] * a.row_bytes
                                          : staged + (size_t)(d - e0) * staged_row;
            buf[u] = NT ? __builtin_nontemporal_load((GPTR(const u32x4))src) : *(GPTR(const u32x4))src;
        }
    };
    auto store = [&](int b, const u32x4(&buf)[SLIDE_U]) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < SLIDE_U; ++u) {
            const int d = b + u * R + lr;
            if (!mine || d >= hi) continue;
            GPTR(u32x4) dst = (GPTR(u32x4))(plane + (size_t)d * a.row_bytes);
            if (NT)
                __builtin_nontemporal_store(buf[u], dst);
            else
                *dst = buf[u];
        }
    };
    // a batch's source indices are loaded two batches ahead, before the rows of
    // the batch in between: loads return in order, so that waiting for the
    // indices never waits for those rows
    int ia[SLIDE_U], ib[SLIDE_U];
    u32x4 A[SLIDE_U], B[SLIDE_U];
    load_idx(lo, ia);
    load_idx(lo + N, ib);
    load(lo, ia, A);
    for (int b = lo; b < hi; b += 2 * N) {
        load_idx(b + 2 * N, ia);
        if (b + N < hi) load(b + N, ib, B);
        store(b, A);
        if (b + N >= hi) break;
        load_idx(b + 3 * N, ib);
        if (b + 2 * N < hi) load(b + 2 * N, ia, A);
        store(b + N, B);
    }
}

// Segments per strip: doubled while the waves are too few to fill the GPU and
// the segments' tails fit the staging area; past SLIDE_FEW waves only while the
// tails stay below 1/32 of the rows.  (512 strips: with 1024-row tails two segments
// took 429 instead of 411 us, with 125-row tails 387 instead of 420; 32 strips of
// a 2-layer cache: in 32 segments 82 us.)
constexpr int SLIDE_FEW = 512, SLIDE_ENOUGH = 1024;
static int slide_segments(int strips, int M, int n_evict, long long row_all, long long area) {
    int s = 1;
    while (strips * s < SLIDE_ENOUGH) {
        const int t = 2 * s;
        const long long tails = (long long)(t - 1) * std::min(n_evict, (M + t - 1) / t);
        if (t > M || tails * row_all > area || (strips * s >= SLIDE_FEW && tails > M / 32)) break;
        s = t;
    }
    return s;
}
// Moves of more bytes than the 256 MiB memory-side cache go past the caches
// (nontemporal): 8192 rows of 64 KiB 249 -> 227 us, 16384 406 -> 382; smaller ones
// through them: 8192 rows of 32 KiB 98 -> 80 us, of 16 KiB 89 -> 73.
constexpr long long SLIDE_CACHED = 256ll << 20;

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Scratch of the indexed eviction for callers that cannot allocate: one copy
// per GPU, held until the process ends.  Host code never passes the array's
// name to a kernel (on the host it is a stand-in, not a device address); it
// passes the address hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) char scratch[KV_NOALLOC_SCRATCH_BYTES];

hipError_t kv_noalloc_scratch(char **out) {
    constexpr int MAX_DEV = 64;
    static std::mutex mu;
    static char *addr[MAX_DEV] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEV) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        addr[dev] = (char *)p;
    }
    *out = addr[dev];
    return hipSuccess;
}

KvWorkspace kv_workspace_layout(int n_layers, int row_bytes, int capacity) {
    KvWorkspace w{};
    const size_t cap = (size_t)capacity;
    size_t off = 0;
    w.offStatus = off;
    off = align256(off + 64);
    w.offPlanes = off;
    off = align256(off + KV_MAX_PLANES * sizeof(char *));
    w.offKeep = off;
    off = align256(off + cap * 4);
    w.offRunStart = off;
    off = align256(off + (cap + 1) * 4);
    w.offRunKey = off;
    off = align256(off + cap * 8);
    w.offRunBkt = off;
    off = align256(off + cap * 4);
    w.offRunTake = off;
    off = align256(off + cap * 4);
    w.offRunFrom = off;
    off = align256(off + cap * 4);
    w.offStage = off;  // tails of the segments of kv_slide
    w.stage_bytes = (size_t)std::min(STAGE_AREA, (long long)capacity * 2 * n_layers * row_bytes);
    off = align256(off + w.stage_bytes);
    w.total = off;
    return w;
}

// ---------------------------------------------------------------------------
// kv_append_indexed: workgroup (t, p) for t < T copies row t of plane p's new
// rows into row s_t of the plane, s_t the t-th entry of the free list
// free_a ++ free_b, 16 bytes a thread; the workgroups of plane 0 also write the
// token's pos, chunk id and slot; workgroups past T (plane 0) copy the rest of
// the free list to free_rest.  Entries outside [0, capacity) are skipped.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void kv_append_kernel(KvAppendLaunch a) {
    const int t = blockIdx.x, p = blockIdx.y;
    auto free_at = [&](int i) { return i < a.na ? a.free_a[i] : a.free_b[i - a.na]; };
    if (t < a.T) {
        const int s = free_at(t);
        if (s < 0 || s >= a.capacity) return;
        const uint4 *src = (const uint4 *)(a.new_rows[p] + (size_t)t * a.row_bytes);
        uint4 *dst = (uint4 *)(a.planes[p] + (size_t)s * a.row_bytes);
        for (int i = threadIdx.x; i < a.row_bytes / 16; i += 256) dst[i] = src[i];
        if (p == 0 && threadIdx.x == 0) {
            a.pos[a.n + t] = a.pos0 + t;
            a.chunk_id[a.n + t] = a.chunk;
            a.slot[a.n + t] = s;
        }
    } else if (p == 0) {
        const int i = (t - a.T) * 256 + threadIdx.x;  // index into the rest of the list
        if (i < a.na + a.nb - a.T) a.free_rest[i] = free_at(a.T + i);
    }
}

hipError_t launch_kv_append(const KvAppendLaunch &p, hipStream_t stream) {
    const int rest = p.na + p.nb - p.T;
    const int gx = p.T + (rest + 255) / 256;
    if (gx == 0) return hipSuccess;
    hipLaunchKernelGGL(kv_append_kernel, dim3(gx, p.n_planes), dim3(256), 0, stream, p);
    return hipGetLastError();
}

hipError_t launch_kv_evict(const KvLaunch &p, hipStream_t stream) {
    char *ws = p.ws;
    KvArgs a;
    a.pos = p.pos;
    a.chunk = p.chunk_id;
    a.scores = p.chunk_scores;
    a.num_chunks = p.num_chunks;
    a.len = p.len;
    a.M = p.M;
    a.n_s = p.n_sink;
    a.n_w = p.n_window;
    a.N = p.n_buckets;
    a.status = (int32_t *)(ws + p.lay.offStatus);
    a.keep = (int32_t *)(ws + p.lay.offKeep);
    a.run_start = (int32_t *)(ws + p.lay.offRunStart);
    a.run_key = (unsigned long long *)(ws + p.lay.offRunKey);
    a.run_bkt = (int32_t *)(ws + p.lay.offRunBkt);
    a.run_take = (int32_t *)(ws + p.lay.offRunTake);
    a.run_from = (int32_t *)(ws + p.lay.offRunFrom);
    a.keep_out = p.keep_out;
    a.slot = p.slot;
    a.free_out = p.free_out;
    a.outcome_out = p.outcome_out;
    a.plane_tab = (char **)(ws + p.lay.offPlanes);
    for (int i = 0; i < KV_MAX_PLANES; ++i) a.planes[i] = i < p.n_planes ? p.planes[i] : nullptr;
    a.n_planes = p.n_planes;
    hipLaunchKernelGGL(kv_select_kernel, dim3(1), dim3(SEL_THREADS), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.slot) return e;  // the indexed variant moves no rows

    if (p.M == 0) return hipSuccess;
    SlideArgs g;
    g.plane_tab = a.plane_tab;
    g.row_bytes = (uint32_t)p.row_bytes;
    g.row_units = (uint32_t)(p.row_bytes / 16);
    g.n_planes = p.n_planes;
    g.M = p.M;
    g.n_evict = p.len - p.M;
    g.pos = p.pos;
    g.chunk = p.chunk_id;
    g.keep = a.keep;
    g.status = a.status;
    g.area = ws + p.lay.offStage;
    // lanes per strip: 128 bytes, or the whole row where it is shorter
    int lpr = 1;
    while (lpr < 8 && lpr < (int)g.row_units) lpr *= 2;
    g.strips = ((int)g.row_units + lpr - 1) / lpr;
    g.segments = slide_segments(p.n_planes * g.strips, p.M, g.n_evict, (long long)p.n_planes * p.row_bytes,
                                (long long)p.lay.stage_bytes);
    g.seg_tail = std::min(g.n_evict, (p.M + g.segments - 1) / g.segments);
    if (g.segments > 1) {
        hipLaunchKernelGGL(kv_stage_tails_kernel, dim3(g.seg_tail, g.segments - 1), dim3(256), 0, stream, g);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    // the first workgroup moves positions and chunk ids
    const dim3 grid(1 + (unsigned)((p.n_planes * g.strips * g.segments + SLIDE_WAVES - 1) / SLIDE_WAVES)), blk(64 * SLIDE_WAVES);
    auto slide = [&](auto lc) {
        constexpr int L = decltype(lc)::value;
        if ((long long)p.M * p.n_planes * p.row_bytes > SLIDE_CACHED)
            hipLaunchKernelGGL((kv_slide_kernel<L, true>), grid, blk, 0, stream, g);
        else
            hipLaunchKernelGGL((kv_slide_kernel<L, false>), grid, blk, 0, stream, g);
    };
    switch (lpr) {
    case 1: slide(std::integral_constant<int, 1>()); break;
    case 2: slide(std::integral_constant<int, 2>()); break;
    case 4: slide(std::integral_constant<int, 4>()); break;
    default: slide(std::integral_constant<int, 8>()); break;
    }
    return hipGetLastError();
}

}  // namespace ds

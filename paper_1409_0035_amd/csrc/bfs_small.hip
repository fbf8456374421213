// Small graphs, unit lengths: one workgroup searches from one sample.
//
// The bit-parallel search of bfs_batched.hip spends two launches a level, and
// on a graph whose arcs and masks sit in a few CUs' reach every launch is a
// chain of dependent round trips with most of the device idle (10,000 nodes,
// 80,000 arcs, 64 samples: 14 level launches of 4-17 us, 181-189 us an
// estimate even when replayed; 72 us this way, the searches 43 and the
// estimates 7 of it).  Here each of the k searches of Sec. 3 of the paper runs in a
// workgroup of its own, with the node's distance (one byte), the visited bits
// and the frontier in LDS, so a level costs a barrier instead of two
// launches, and one launch does all searches.  The same workgroup then has
// everything Algorithm 1 keeps per sample -- the sample distance matrix's row,
// the level histogram, its tail tables, S(c_i) -- and writes it; a second
// launch (k_small_estimate) evaluates every node.
//
// What bounds it: the latency of a level (four barriers of 16 waves, frontier,
// row bounds, arc ids; about 2.5 us) and, as the arcs grow, one CU's rate of arc visits: every
// sample reads the arcs for itself, where the bit-parallel search reads them
// once for 64 samples.  The host's rule (small_search_fits) draws that line.
//
// A level pushes from its frontier (a list in LDS whose arcs are dealt to the
// threads by a prefix sum of the degrees, so a hub costs what its arcs cost)
// while the frontier's arcs are fewer than a pull would read; otherwise it pulls:
// a lane per unvisited node reads its arcs four at a time until one of them
// ends at a node of an earlier level, which the triangle argument of
// bfs_batched.hip makes the previous level.  Lanes left after 64 arcs finish
// their rows together.
#include "internal.h"

#include <algorithm>

namespace ccg {

namespace {

constexpr int kSB = 1024;         // threads of a search
constexpr int kSWaves = kSB / 64;
constexpr int32_t kQCap = 4096;   // frontier entries a push level can take
constexpr int kPerT = kQCap / kSB;
constexpr size_t kLdsBytes = 160 * 1024;
constexpr int kU = 4;             // 64-node chunks a wave pulls for at a time
constexpr uint8_t kFar = 0xFF;
constexpr int32_t kMaxLevel = 254;

typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));

struct SearchLds {
    uint8_t* dist;      // [npad]
    uint32_t* vis;      // [npad / 32]
    int32_t* q;         // [2][qcap] the frontier, by level parity
    uint32_t* first;    // [qcap] a frontier node's first arc, less the arcs of the nodes before it
    uint32_t* upto;     // [qcap] the arcs of the frontier up to and with the node
    int32_t* hist;      // [256]
    int32_t* cnt;       // [2] nodes found, by level parity
    uint32_t* part;     // [kSWaves]
};

// The arcs of one direction: in memory, or copied to LDS with two-byte ids.
struct ArcsGlobal {
    const uint32_t* __restrict__ rp;
    const int32_t* __restrict__ col;
    uint32_t arcs;
    __device__ __forceinline__ uint32_t row(int32_t v) const { return rp[v]; }
    __device__ __forceinline__ int32_t at(uint32_t t) const { return col[t]; }
    __device__ __forceinline__ i32x4 four(uint32_t b, uint32_t e) const {  // arcs b .. b + 3; past e anything
        i32x4 x = i32x4{0, 0, 0, 0};
        if (b + 4 <= arcs) {
            x = *(const i32x4*)(col + b);
        } else {  // the array's last arcs
            for (int q = 0; q < 4; q++)
                if (b + q < e) x[q] = col[b + q];
        }
        return x;
    }
};
struct ArcsLds {
    const uint32_t* rp;
    const uint16_t* col;
    uint32_t arcs;
    __device__ __forceinline__ uint32_t row(int32_t v) const { return rp[v]; }
    __device__ __forceinline__ int32_t at(uint32_t t) const { return col[t]; }
    __device__ __forceinline__ i32x4 four(uint32_t b, uint32_t e) const {
        i32x4 x;
#pragma unroll
        for (int q = 0; q < 4; q++) x[q] = col[min(b + q, e - 1)];
        return x;
    }
};

// One breadth-first search from src by the whole workgroup.  Returns the last
// level that found a node; *status: 0 every node reached, 1 some not, 2 more
// than 254 levels.
template <typename Arcs>
__device__ __forceinline__ int32_t small_bfs(const Arcs& in, const Arcs& out, int32_t n, int32_t npad, int32_t qcap,
                                             int32_t src, const SearchLds& S, int64_t* scanned, int32_t* status) {
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    for (int t = tid; t < npad / 4; t += kSB) ((uint32_t*)S.dist)[t] = 0xFFFFFFFFu;
    for (int t = tid; t < npad / 32; t += kSB) S.vis[t] = 0;
    if (tid < 256) S.hist[tid] = 0;
    __syncthreads();
    if (tid == 0) {
        S.dist[src] = 0;
        S.vis[src >> 5] = 1u << (src & 31);
        S.q[0] = src;
        S.cnt[0] = 1;
        S.cnt[1] = 0;
        S.hist[0] = 1;
    }
    int32_t visited = 1;
    uint32_t seen = 0;   // arcs visited by this thread
    uint32_t known = 0;  // arcs of the nodes found so far, but for levels longer than their list
    const int32_t nchunks = npad / 64;
    for (int32_t level = 1;; level++) {
        const int cur = (level - 1) & 1, nxt = level & 1;
        __syncthreads();
        const int32_t nf = S.cnt[cur];
        // a frontier that its list holds: where each node's arcs lie among all of them
        uint32_t mf = 0;
        if (nf <= qcap) {
            uint32_t b[kPerT] = {}, d[kPerT] = {}, own = 0, upto = 0;
            const bool some = wave * 64 * kPerT < nf;  // waves past the frontier's end have nothing here
            if (some) {
#pragma unroll
                for (int r = 0; r < kPerT; r++) {
                    const int32_t at = tid * kPerT + r;
                    b[r] = d[r] = 0;
                    if (at < nf) {
                        const int32_t v = S.q[cur * qcap + at];
                        b[r] = out.row(v);
                        d[r] = out.row(v + 1);
                    }
                }
#pragma unroll
                for (int r = 0; r < kPerT; r++) {
                    d[r] -= b[r];
                    own += d[r];
                }
                upto = own;  // inclusive over the wave
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t o = (uint32_t)__shfl_up((int)upto, off);
                    if (lane >= off) upto += o;
                }
            }
            if (lane == 63) S.part[wave] = upto;
            __syncthreads();
            const int nw = (nf + 64 * kPerT - 1) / (64 * kPerT);
            for (int w = 0; w < nw; w++) {
                const uint32_t x = S.part[w];
                mf += x;
                if (w < wave) upto += x;
            }
            upto -= own;
            if (some) {
#pragma unroll
                for (int r = 0; r < kPerT; r++) {
                    const int32_t at = tid * kPerT + r;
                    if (at < nf) {
                        S.first[at] = b[r] - upto;
                        upto += d[r];
                        S.upto[at] = upto;
                    }
                }
            }
            __syncthreads();
        }
        // push while the frontier's arcs are few against what a pull would
        // scan, or so few that a trip or two of the workgroup covers them.  A
        // pull reads a node's arcs until one ends at a node found before: about
        // arcs / known of them where arcs end anywhere, but no more than the
        // node has (arcs / n), and four at the least.  (A pull taken for one
        // trip of four arcs a node, which holds where hubs were found early,
        // read most of a flat random graph's arcs in its widest level: 49,000
        // nodes of 40 arcs, 64 samples 339 -> 193 us; R-MAT scale 16 217 ->
        // 177 us.)
        known += mf;
        const float four = 4.0f * (float)max((uint32_t)n, known);
        const bool push = nf <= qcap && (mf <= 4 * kSB || (float)mf * four < (float)(n - visited) * fmaxf((float)out.arcs, four));
        if (push) {
            int32_t top = 1;
            while (top < nf) top <<= 1;
            for (uint32_t x0 = 4 * tid; x0 - 4 * lane < mf; x0 += 4 * kSB) {  // wave-uniform trips
                // the frontier node of the thread's first arc, the first whose
                // count passes it; the three arcs after it mostly share its row
                int32_t lo = 0, u[4];
                bool mine[4];
                if (x0 < mf) {
                    lo = -1;
                    for (int32_t step = top; step > 0; step >>= 1) {
                        const int32_t at = lo + step;
                        if (at < nf && S.upto[at] <= x0) lo = at;
                    }
                    lo++;
                }
                uint32_t end = x0 < mf ? S.upto[lo] : 0, base = x0 < mf ? S.first[lo] : 0;
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const uint32_t x = x0 + r;
                    u[r] = -1;
                    if (x < mf) {
                        while (x >= end) {
                            end = S.upto[++lo];
                            base = S.first[lo];
                        }
                        u[r] = out.at(base + x);
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; r++) mine[r] = u[r] >= 0 && S.dist[u[r]] == kFar;
#pragma unroll
                for (int r = 0; r < 4; r++)
                    if (mine[r]) {
                        const uint32_t bit = 1u << (u[r] & 31);
                        mine[r] = !(atomicOr(&S.vis[u[r] >> 5], bit) & bit);
                        if (mine[r]) S.dist[u[r]] = (uint8_t)level;
                    }
                uint64_t m[4];
                int32_t total = 0;
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    m[r] = __ballot(mine[r]);
                    total += (int32_t)__popcll(m[r]);
                }
                if (total) {
                    int32_t put = 0;
                    if (lane == 0) put = atomicAdd(&S.cnt[nxt], total);
                    put = readlane32(put, 0);
#pragma unroll
                    for (int r = 0; r < 4; r++) {
                        const int32_t at = put + (int32_t)__popcll(m[r] & lanemask_lt());
                        if (mine[r] && at < qcap) S.q[nxt * qcap + at] = u[r];
                        put += (int32_t)__popcll(m[r]);
                    }
                }
            }
            if (tid == 0) seen += mf;
        } else {
            for (int32_t c0 = wave; c0 < nchunks; c0 += kSWaves * kU) {
                int32_t v[kU];
                uint32_t b[kU], e[kU];
                bool open[kU], found[kU];
                bool any = false;
#pragma unroll
                for (int r = 0; r < kU; r++) {
                    const int32_t c = c0 + kSWaves * r;
                    v[r] = c * 64 + lane;
                    open[r] = c < nchunks && v[r] < n && S.dist[v[r]] == kFar;
                    found[r] = false;
                    b[r] = e[r] = 0;
                    any = any || open[r];
                }
                if (!__ballot(any)) continue;
#pragma unroll
                for (int r = 0; r < kU; r++)
                    if (open[r]) {
                        b[r] = in.row(v[r]);
                        e[r] = in.row(v[r] + 1);
                    }
#pragma unroll
                for (int r = 0; r < kU; r++) open[r] = open[r] && b[r] < e[r];
                i32x4 x[kU];
#pragma unroll
                for (int r = 0; r < kU; r++) {
                    x[r] = i32x4{0, 0, 0, 0};
                    if (open[r]) x[r] = in.four(b[r], e[r]);
                }
#pragma unroll
                for (int r = 0; r < kU; r++) {
                    bool hit = false;
#pragma unroll
                    for (int q = 0; q < 4; q++) hit |= (S.dist[x[r][q]] < level) & (b[r] + q < e[r]);
                    if (open[r]) {
                        seen += min(4u, e[r] - b[r]);
                        b[r] += 4;
                        found[r] = hit;
                        open[r] = !hit && b[r] < e[r];
                    }
                }
                // rows without a hit there: 16 arcs a trip, so that a row's
                // cache line is used while it is there
#pragma unroll
                for (int r = 0; r < kU; r++) {
                    for (int trip = 0; trip < 4 && __ballot(open[r]); trip++) {
                        if (open[r]) {
                            i32x4 y[4];
#pragma unroll
                            for (int q = 0; q < 4; q++) {
                                y[q] = i32x4{0, 0, 0, 0};
                                if (b[r] + 4 * q < e[r]) y[q] = in.four(b[r] + 4 * q, e[r]);
                            }
                            bool hit = false;
#pragma unroll
                            for (int q = 0; q < 16; q++)
                                hit |= (S.dist[y[q / 4][q % 4]] < level) & (b[r] + q < e[r]);
                            seen += min(16u, e[r] - b[r]);
                            b[r] += 16;
                            found[r] = hit;
                            open[r] = !hit && b[r] < e[r];
                        }
                    }
                }
#pragma unroll
                for (int r = 0; r < kU; r++) {  // long rows: the rest by the whole wave
                    uint64_t m = __ballot(open[r]);
                    while (m) {
                        const int s = __ffsll((unsigned long long)m) - 1;
                        m &= m - 1;
                        const uint32_t bb = (uint32_t)readlane32((int)b[r], s), ee = (uint32_t)readlane32((int)e[r], s);
                        bool hit = false;
                        for (uint32_t t = bb; t < ee && !hit; t += 128) {
                            const uint32_t t0 = t + lane, t1 = t0 + 64;
                            const bool h = (t0 < ee && S.dist[in.at(t0)] < level) || (t1 < ee && S.dist[in.at(t1)] < level);
                            hit = __ballot(h) != 0;
                            if (lane == 0) seen += min(128u, ee - t);
                        }
                        if (lane == s) found[r] = hit;
                    }
                    // the chunk's visited bits have this one writer
                    const uint64_t f = __ballot(found[r]);
                    if (f) {
                        if (lane == 0) {
                            uint64_t* w = (uint64_t*)S.vis + (c0 + kSWaves * r);
                            *w |= f;
                        }
                        if (found[r]) S.dist[v[r]] = (uint8_t)level;
                        const int at = wave_append(&S.cnt[nxt], found[r]);
                        if (at >= 0 && at < qcap) S.q[nxt * qcap + at] = v[r];
                    }
                }
            }
        }
        __syncthreads();
        const int32_t nn = S.cnt[nxt];
        if (tid == 0) {  // read again only after the next barrier
            S.hist[level] = nn;
            S.cnt[cur] = 0;
        }
        visited += nn;
        if (nn == 0 || visited == n || level == kMaxLevel) {
            *scanned += seen;
            *status = visited == n ? 0 : (nn == 0 ? 1 : 2);
            return nn == 0 ? level - 1 : level;
        }
    }
}

// A direction's arcs copied to LDS (two-byte ids), by the whole workgroup.
__device__ __forceinline__ void copy_arcs(const uint32_t* __restrict__ rp, const int32_t* __restrict__ col, int32_t n,
                                          uint32_t arcs, uint32_t* lrp, uint16_t* lcol) {
    for (int t = threadIdx.x; t <= n; t += kSB) lrp[t] = rp[t];
    for (uint32_t t = threadIdx.x; t < arcs; t += kSB) lcol[t] = (uint16_t)col[t];
}

template <bool RT, bool LA>
__global__ __launch_bounds__(kSB) void k_small_search(SmallArgs a, SmallSamples ss) {
    extern __shared__ uint8_t lds[];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int32_t i = blockIdx.x, n = a.n, k = a.k, npad = a.npad, qcap = a.qcap;
    const uint64_t t0 = wall_clock64();
    const int32_t src = ss.ids[i];
    int64_t scanned = 0;
    SearchLds S;
    S.dist = lds;
    S.vis = (uint32_t*)(lds + npad);
    S.q = (int32_t*)(lds + npad + npad / 8);
    S.first = (uint32_t*)(S.q + 2 * qcap);
    S.upto = S.first + qcap;
    S.hist = (int32_t*)(S.upto + qcap);
    S.cnt = S.hist + 256;
    S.part = (uint32_t*)(S.cnt + 2);
    uint32_t* lrp = S.part + kSWaves;          // LA: the row bounds and the arcs
    uint16_t* lcol = (uint16_t*)(lrp + n + 1);
    auto search = [&](bool reverse, int32_t* st) {
        if constexpr (LA) {
            const ArcsLds out{lrp, lcol, a.arcs};
            const int32_t* c = reverse ? a.in_col : a.out_col;
            copy_arcs(reverse ? a.in_rp : a.out_rp, c, n, a.arcs, lrp, lcol);
            if constexpr (RT) {
                // the other direction's arcs follow
                uint32_t* lrp2 = (uint32_t*)(lcol + (a.arcs + 1) / 2 * 2);
                uint16_t* lcol2 = (uint16_t*)(lrp2 + n + 1);
                const ArcsLds in{lrp2, lcol2, a.arcs};
                copy_arcs(reverse ? a.out_rp : a.in_rp, reverse ? a.out_col : a.in_col, n, a.arcs, lrp2, lcol2);
                return small_bfs(in, out, n, npad, qcap, src, S, &scanned, st);
            } else {
                return small_bfs(out, out, n, npad, qcap, src, S, &scanned, st);
            }
        } else {
            const ArcsGlobal f{a.out_rp, a.out_col, a.arcs}, r{a.in_rp, a.in_col, a.arcs};
            return reverse ? small_bfs(f, r, n, npad, qcap, src, S, &scanned, st)
                           : small_bfs(r, f, n, npad, qcap, src, S, &scanned, st);
        }
    };
    int32_t* s_row = S.q;  // [k], k <= n: the sample distance row, once the searches are over
    int32_t status = 0;
    int32_t ecc = search(false, &status);
    int32_t levels = ecc;
    uint32_t* row = (uint32_t*)(a.Dt + (int64_t)i * npad);
    __syncthreads();
    if constexpr (RT) {
        for (int t = tid; t < npad / 4; t += kSB) row[t] = ((const uint32_t*)S.dist)[t];
        __syncthreads();
        int32_t st2 = 0;
        const int32_t e2 = search(true, &st2);
        levels += e2;
        if (status == 0) status = st2;
        if (status == 0 && ecc + e2 > kMaxLevel) status = 2;  // a sum may not fit a byte
        ecc += e2;
        __syncthreads();
        // summed rows (each thread reads back its own words) and their
        // histogram, in copies by lane (the lanes of a wave agree on few
        // values) where the frontier was
        const int nc = min(16, qcap / 64);
        int32_t* copies = S.q;
        for (int t = tid; t < 256 * nc; t += kSB) copies[t] = 0;
        __syncthreads();
        if (status == 0) {
            for (int base = 0; base < npad / 4; base += kSB) {
                const int t = base + tid;
                const bool in = t < npad / 4;
                const uint32_t f = in ? row[t] : 0, r = in ? ((const uint32_t*)S.dist)[t] : 0;
                uint32_t sum = 0;
#pragma unroll
                for (int q = 0; q < 4; q++) {
                    const bool real = in && t * 4 + q < n;
                    const uint32_t dv = real ? ((f >> (8 * q)) & 0xFF) + ((r >> (8 * q)) & 0xFF) : kFar;
                    sum |= dv << (8 * q);
                    if (real) atomicAdd(&copies[dv * nc + (lane & (nc - 1))], 1);
                }
                if (in) {
                    row[t] = sum;
                    ((uint32_t*)S.dist)[t] = sum;
                }
            }
        }
        __syncthreads();
        if (tid < 256) {
            int32_t c = 0;
            for (int q = 0; q < nc; q++) c += copies[tid * nc + q];
            S.hist[tid] = c;
        }
        __syncthreads();
    } else {
        for (int t = tid; t < npad / 4; t += kSB) row[t] = ((const uint32_t*)S.dist)[t];
    }
    // row i of the sample distance matrix; the samples leave the histogram
    for (int j = tid; j < k; j += kSB) {
        const uint8_t d = S.dist[ss.ids[j]];
        a.dmat_c[(int64_t)i * k + j] = d;
        s_row[j] = d;
        atomicAdd(&S.hist[d], -1);
    }
    __syncthreads();
    // L masks of i as a pivot, Lmask[i][t] = {j : d(c_i, c_j) <= t}, up to the row's largest entry
    int32_t rmax = 0, rsum = 0;
    for (int j = lane; j < k; j += 64) {
        rmax = max(rmax, s_row[j]);
        rsum += s_row[j];
    }
    rsum = wave_sum32(rsum);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) rmax = max(rmax, __shfl_xor(rmax, off));
    const int W = (k + 63) / 64;
    if (status == 0)
        for (int t = wave; t <= rmax; t += kSWaves)
            for (int w = 0; w < W; w++) {
                const int j = w * 64 + lane;
                const uint64_t m = __ballot(j < k && s_row[j] <= t);
                if (lane == 0) a.lmask[((int64_t)i * kSmallT + t) * W + w] = m;
            }
    // tail tables T_cnt[t] = sum_{d >= t} h[d], T_sum[t] = sum_{d >= t} d h[d] over unsampled nodes
    if (tid < kSmallT) {
        int32_t c = 0;
        int64_t sm = 0;
        for (int d = min(ecc, kMaxLevel); d >= tid; d--) {
            const int32_t h = S.hist[d];
            c += h;
            sm += (int64_t)d * h;
        }
        a.Tcnt[(int64_t)i * kSmallT + tid] = c;
        a.Tsum[(int64_t)i * kSmallT + tid] = sm;
        if (tid == 0) {
            a.src_sum[i] = sm + rsum;  // S(c_i)
            a.rmax[i] = rmax;
            a.status[i] = status;
        }
    }
    scanned = wave_sum64(scanned);
    __syncthreads();
    // a level reads an arc once at most: 2 x 254 levels of 2^21 arcs fit 32 bits
    if (lane == 0) S.part[wave] = (uint32_t)scanned;
    __syncthreads();
    if (tid == 0) {
        uint32_t s = 0;
        for (int w = 0; w < kSWaves; w++) s += S.part[w];
        // one 16-byte store to the host's memory
        *(uint4*)(a.rec + i) = make_uint4((uint32_t)status | (uint32_t)ecc << 4 | (uint32_t)levels << 16, s,
                                          (uint32_t)t0, (uint32_t)wall_clock64());
    }
}

// Every node's estimates (Sec. 2, Eqs. (5), (6)) from the searches' rows and
// tables: a workgroup takes 64 nodes, wave w the samples 64 w .. 64 w + 63,
// whose distances it keeps packed in 16 registers for both passes (pivot and
// sum, then the sum over L cap C by the pivot's mask); wave 0 finishes.  The
// integers and the order of double operations are those of k_estimate_bits.
template <int W>
__global__ __launch_bounds__(64 * W) void k_small_estimate(SmallArgs a, SmallOut o, SmallSamples ss) {
    __shared__ uint32_t s_key[W][64], s_sum[W][64], s_cnt[W][64], s_lc[W][64];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int32_t n = a.n, k = a.k;
    bool bad = false;
#pragma unroll
    for (int j = 0; j < W; j++) bad = bad || a.status[min(64 * j + lane, k - 1)] != 0;
    const int64_t gid = (int64_t)blockIdx.x * (64 * W) + tid, all = (int64_t)gridDim.x * (64 * W);
    const int32_t v = blockIdx.x * 64 + lane;  // below npad
    const int nb = min(64, k - 64 * w);
    const uint8_t* col = a.Dt + (int64_t)(64 * w) * a.npad + v;
    // all 64 loads go out together: past the last sample they read it again
    uint8_t raw[64];
#pragma unroll
    for (int i = 0; i < 64; i++) raw[i] = col[(uint32_t)min(i, nb - 1) * (uint32_t)a.npad];
    uint32_t x[16];
#pragma unroll
    for (int q = 0; q < 16; q++)
        x[q] = (uint32_t)raw[4 * q] | (uint32_t)raw[4 * q + 1] << 8 | (uint32_t)raw[4 * q + 2] << 16 |
               (uint32_t)raw[4 * q + 3] << 24;
    if (__ballot(bad)) return;  // a search failed: every output is left alone (the same in every wave)
    uint32_t key = 0xFFFFFFFFu, sum = 0;
#pragma unroll
    for (int q = 0; q < 16; q++)
#pragma unroll
        for (int b = 0; b < 4; b++)
            if (4 * q + b < nb) {
                const uint32_t d = (x[q] >> (8 * b)) & 0xFF;
                key = min(key, (d << 8) | (uint32_t)(64 * w + 4 * q + b));  // ties to the lowest sample
                sum += d;
            }
    s_key[w][lane] = key;
    s_sum[w][lane] = sum;
    __syncthreads();
    int64_t total = 0;
#pragma unroll
    for (int u = 0; u < W; u++) {
        key = min(key, s_key[u][lane]);
        total += s_sum[u][lane];
    }
    const bool valid = v < n;
    const int64_t ov = valid ? a.orig[v] : 0;
    const int32_t p = valid ? (int32_t)(key & 0xFF) : 0, delta = valid ? (int32_t)(key >> 8) : 0;
    int64_t thr = (int64_t)delta * a.ed / a.en;  // L: d(c(v), u) <= floor(Delta / eps)
    const int64_t tix = thr + 1;
    thr = min(thr, (int64_t)a.rmax[p]);
    const uint64_t m = a.lmask[((int64_t)p * kSmallT + thr) * W + w];
    uint32_t lc = 0;
#pragma unroll
    for (int q = 0; q < 16; q++) {
        const uint32_t four = (uint32_t)(m >> (4 * q)) & 0xF;
        const uint32_t bytes = ((four * 0x00204081u) & 0x01010101u) * 0xFFu;  // a byte mask of the four bits
        lc = __builtin_amdgcn_sad_u8(x[q] & bytes, 0u, lc);
    }
    s_cnt[w][lane] = (uint32_t)__popcll(m);
    s_lc[w][lane] = lc;
    __syncthreads();
    if (o.dmat)
        for (int64_t t = gid; t < (int64_t)k * k; t += all) o.dmat[t] = a.dmat_c[t];
    if (gid < k) {
        if (o.src_sum) o.src_sum[gid] = a.src_sum[gid];
        if (o.samples) o.samples[gid] = ss.caller[gid];
    }
    if (!valid) return;
    if (o.D) {  // int32 rows at the caller's ids
        int32_t* dst = o.D + ov * k + 64 * w;
#pragma unroll
        for (int q = 0; q < 16; q++)
#pragma unroll
            for (int b = 0; b < 4; b++)
                if (4 * q + b < nb) dst[4 * q + b] = (int32_t)((x[q] >> (8 * b)) & 0xFF);
    }
    if (o.rows) {  // byte rows in internal order, for the error pass
        uint8_t* dst = o.rows + (int64_t)v * k + 64 * w;
#pragma unroll
        for (int q = 0; q < 16; q++)
#pragma unroll
            for (int b = 0; b < 4; b++)
                if (4 * q + b < nb) dst[4 * q + b] = (uint8_t)(x[q] >> (8 * b));
    }
    if (w != 0) return;
    if (o.sidx) o.sidx[v] = delta == 0 ? p : -1;
    int64_t lcsum = 0, lcnum = 0;
#pragma unroll
    for (int u = 0; u < W; u++) {
        lcsum += s_lc[u][lane];
        lcnum += s_cnt[u][lane];
    }
    const int64_t LIM = (int64_t)1 << 53;
    double hyb, samp;
    int64_t piv, pub;
    bool ovf;
    if (delta == 0) {  // lengths are positive: v is the sample p
        const int64_t Sp = a.src_sum[p];
        hyb = samp = (double)Sp;
        piv = pub = Sp;
        ovf = Sp >= LIM;
    } else {
        int64_t hnum = 0, hsum = 0;
        if (tix < kSmallT) {
            hnum = a.Tcnt[(int64_t)p * kSmallT + tix];
            hsum = a.Tsum[(int64_t)p * kSmallT + tix];
        }
        const int64_t lnum = ((int64_t)n - 1) - hnum - ((int64_t)k - lcnum);
        const int64_t h = hsum + (total - lcsum);
        int64_t t1 = 0, t2 = 0, N = 0, s2 = 0;
        ovf = __builtin_mul_overflow(h, lcnum, &t1) || __builtin_mul_overflow(lcsum, lnum, &t2) ||
              __builtin_add_overflow(t1, t2, &N) || N >= LIM || lcnum < 1 || lnum < lcnum;
        hyb = (double)N / (double)lcnum;
        ovf = ovf || __builtin_mul_overflow((int64_t)n - 1, total, &s2) || s2 >= LIM;
        samp = (double)s2 / (double)k;
        piv = a.src_sum[p];
        pub = piv + ((int64_t)n - 1) * delta;
    }
    if (o.S_hyb) o.S_hyb[ov] = hyb;
    if (o.S_samp) o.S_samp[ov] = samp;
    if (o.S_piv) o.S_piv[ov] = piv;
    if (o.S_pub) o.S_pub[ov] = pub;
    if (o.pivot) o.pivot[ov] = p;
    if (o.delta) o.delta[ov] = delta;
    if (o.sampsum) o.sampsum[ov] = total;
    if (ovf) __hip_atomic_store(&a.flags->overflow, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    if (lane == 0)  // any late block's stamp tells when the estimates were done
        __hip_atomic_store(a.stamps + (blockIdx.x % kSmallStamps), (uint32_t)wall_clock64(), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_SYSTEM);
}

size_t small_lds(int32_t npad, int32_t qcap) {
    return (size_t)npad + npad / 8 + sizeof(int32_t) * (4 * (size_t)qcap + 256 + 2 + kSWaves);
}

template <bool RT, bool LA>
void launch_search(hipStream_t st, const SmallArgs& a, const SmallSamples& ss, size_t lds) {
    // the limit is the kernel's, for all threads: every call sets the same value
    if (lds > 65536)
        CCG_HIP(hipFuncSetAttribute((const void*)k_small_search<RT, LA>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)kLdsBytes));
    hipLaunchKernelGGL((k_small_search<RT, LA>), dim3((unsigned)a.k), dim3(kSB), lds, st, a, ss);
}

}  // namespace

void small_estimate(hipStream_t st, SmallArgs a, const SmallOut& o, const SmallSamples& ss, bool round_trip) {
    a.qcap = std::max(std::min(kQCap, a.npad), kSmallSamples);
    const size_t lds = small_lds(a.npad, a.qcap);
    // arcs that fit LDS beside the search's state are copied there: a level
    // then waits for no memory
    const size_t one = sizeof(uint32_t) * ((size_t)a.n + 1) + sizeof(uint16_t) * (((size_t)a.arcs + 1) / 2 * 2);
    const size_t copied = lds + one * (round_trip ? 2 : 1);
    const bool la = copied <= kLdsBytes;
    if (round_trip) la ? launch_search<true, true>(st, a, ss, copied) : launch_search<true, false>(st, a, ss, lds);
    else la ? launch_search<false, true>(st, a, ss, copied) : launch_search<false, false>(st, a, ss, lds);
    const dim3 grid((unsigned)(a.npad / 64));
    switch ((a.k + 63) / 64) {
        case 1: hipLaunchKernelGGL((k_small_estimate<1>), grid, dim3(64), 0, st, a, o, ss); break;
        case 2: hipLaunchKernelGGL((k_small_estimate<2>), grid, dim3(128), 0, st, a, o, ss); break;
        case 3: hipLaunchKernelGGL((k_small_estimate<3>), grid, dim3(192), 0, st, a, o, ss); break;
        default: hipLaunchKernelGGL((k_small_estimate<4>), grid, dim3(256), 0, st, a, o, ss); break;
    }
    CCG_HIP(hipGetLastError());
}

}  // namespace ccg

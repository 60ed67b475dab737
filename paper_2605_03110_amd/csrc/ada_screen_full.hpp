// The full selection of one long sequence from the graph of near pairs (ada_screen.hpp), with every token's largest
// correlation.  Included by ada_kernels.hip after ada_gram_dma.hpp.
//
// The set follows from clusters and edges alone.  A token's largest |cos| to an earlier token does as well, up to the few
// products that compete for it: a token of a cluster is closer to its pivot than any pair that is no candidate can be, so
// its maximum lies among the earlier members of its cluster (and the unexplained candidates multiplied out); only a token
// that is in no earlier token's cluster, a HEAD, has to meet all earlier tokens.  With K centres among T tokens heads come
// early -- a new centre is met for the first time after about K tokens -- so their rows of the triangle are short:
// 0.5% of it at T = 8192, K = 400, a third at K = T / 2.
//
//   k_screen_sort  one workgroup: the set; the members of clusters of two and more, cluster by cluster; the heads;
//                  and the tiles that follow from both, or the word that sends the call to the full Gram instead.
//   k_screen_gram  tiles of two kinds: the members' list against itself, a block against itself and the blocks that its first
//                  cluster reaches back to (products between clusters are wasted but not wrong: every product is one of
//                  the row's; where there are many members a block ends between clusters), and
//                  the heads against the tokens before them.  64 x 64; 128 x 128 for the heads where there are many.
#pragma once

// Words of the work list (in the unit's memory for pivots, which nobody reads any more).  SW_FIRST: where a block of members starts and,
// from bit 16 on, the first block of the cluster that it starts in.  Two blocks that follow each other hold at least 65 members, but for the
// last one of each lane's (sort_blocks).
constexpr int SORT_LANE = 512;                                // members a lane of sort_blocks goes through
constexpr int SORT_MEMBER_BLOCKS = FUSED_MAX_T / 32 + FUSED_MAX_T / SORT_LANE, SORT_HEAD_BLOCKS = FUSED_MAX_T / 64;
static_assert(2 * FUSED_MAX_T / 65 + FUSED_MAX_T / SORT_LANE <= SORT_MEMBER_BLOCKS && FUSED_MAX_T / SORT_LANE <= 64, "blocks of members, a lane per 512 of them");
enum { SW_BLOCKS = 0, SW_HEADS = 1, SW_TILES = 2, SW_TILES128 = 3, SW_FIRST = 16, SW_PRE = SW_FIRST + SORT_MEMBER_BLOCKS + 1,
       SW_PRE128 = SW_PRE + SORT_MEMBER_BLOCKS + SORT_HEAD_BLOCKS + 1, SW_WORDS = SW_PRE128 + SORT_HEAD_BLOCKS / 2 + 1 };
constexpr int SCREEN_FULL_MIN_T = 1500;                       // the work list fits the pivots' memory
static_assert(SW_WORDS <= SCREEN_FULL_MIN_T && FUSED_MAX_T < 1 << 15 && SORT_MEMBER_BLOCKS + SORT_HEAD_BLOCKS < 1024, "work list");
// Pairs inside clusters per token above which their tiles are no saving (clusters of about 128 and more)
constexpr uint32_t SCREEN_FULL_PAIRS = 64;

struct ScreenFullParams {
    ScreenParams s;            // one unit
    int want_gamma, greedy, big_tiles;   // big_tiles: 64 x 64 tiles of heads from which on they are cut into 128 x 128
    float most_heads;          // share of the triangle above which the heads' tiles are no saving
    int whole_from;            // members from which on their blocks end between clusters, see k_screen_sort
    int ntile, lanes, f32;     // of the unexplained candidates, see screen_rest_tiles
    int32_t* gate;             // out: 1 = the graph does not decide, the launches behind run the full Gram
    uint8_t* mask;             // may be NULL
    int32_t* idx;              // may be NULL
    int32_t* counts;
    unsigned long long* ops;   // may be NULL
};

struct ScreenLists { int32_t *work, *member, *head; };
__device__ inline ScreenLists screen_full_lists(const ScreenParams& p, const ScreenUnit& U) {
    return {reinterpret_cast<int32_t*>(p.area + U.o_piv), reinterpret_cast<int32_t*>(p.area + U.o_size),
            reinterpret_cast<int32_t*>(p.area + U.o_rho)};
}

constexpr int SCREEN_SORT_THREADS = 1024;
inline int screen_sort_lds(int T) {                           // counts (4 bytes), clusters and members (2 bytes each)
    return std::max((T + 63) / 64 * 64 * 8, SCREEN_SORT_THREADS / 256 * (int)sizeof(RestTile));
}

// Exclusive sums of two words over the workgroup (sums: one int2 per wave, not used before).
__device__ inline int2 screen_scan(int2 v, int2* total, int2* sums) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int2 inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(inc.x, o, 64), y = __shfl_up(inc.y, o, 64);
        if (lane >= o) { inc.x += x; inc.y += y; }
    }
    if (lane == 63) sums[wave] = inc;
    screen_barrier();
    int2 before = {0, 0}, all = {0, 0};
#pragma unroll
    for (int w = 0; w < SCREEN_SORT_THREADS / 64; ++w) {
        const int2 x = sums[w];
        if (w < wave) { before.x += x.x; before.y += x.y; }
        all.x += x.x;
        all.y += x.y;
    }
    *total = all;
    return int2{before.x + inc.x - v.x, before.y + inc.y - v.y};
}

// What a cluster's count becomes: the next free place in the list, and whether the cluster lies in several blocks.
constexpr uint32_t SORT_PLACED = 0x80000000u, SORT_LARGE = 0x40000000u, SORT_PLACE = 0x3FFFFFFFu;

// The last cluster that starts at or before member p (edge: a bit where a cluster starts; 0 is a start, if there is any).
__device__ inline int sort_start(const unsigned long long* edge, int p) {
    int w = p >> 6;
    unsigned long long m = edge[w] & (~0ull >> (63 - (p & 63)));
    while (m == 0ull && w > 0) m = edge[--w];
    return m ? w * 64 + 63 - __clzll((long long)m) : 0;
}

// Cuts the members' list into blocks of up to 64, between clusters where it can be (one wave; first, blocks: out, see
// SW_FIRST).  From a block's start on, the next one starts at the last cluster that starts within 64 members.  Each lane goes
// through about 512 members like this, from a cluster's start to one, so a chain of ten steps takes the place of one of
// mem / 60; half a block more per lane is the price.  (A larger cluster starts a block, as no other starts within the 64
// behind it.)
__device__ inline void sort_blocks(const unsigned long long* edge, int mem, uint32_t* first, int* blocks) {
    const int lane = threadIdx.x & 63;
    const int lo = lane * SORT_LANE < mem ? sort_start(edge, lane * SORT_LANE) : mem,
              up = (lane + 1) * SORT_LANE < mem ? sort_start(edge, (lane + 1) * SORT_LANE) : mem;
    auto walk = [&](auto emit) {
        int n = 0, of = 0;                                    // blocks so far, the first one of the cluster at hand
        bool starts = true;                                   // p is a cluster's start
        for (int p = lo; p < up;) {
            if (starts) of = n;
            emit(n, p, of);
            ++n;
            if (p + 64 >= up) break;
            const int w = p >> 6, b = p & 63;                 // the starts behind p, up to p + 64, as bits 0 .. 63
            const unsigned long long m = (b < 63 ? edge[w] >> (b + 1) : 0ull) | edge[w + 1] << (63 - b);
            starts = m != 0ull;
            p += starts ? 64 - __clzll((long long)m) : 64;
        }
        return n;
    };
    const int n = walk([](int, int, int) {});
    int inc = n;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(inc, o, 64);
        if (lane >= o) inc += x;
    }
    const int before = inc - n;
    walk([&](int k, int p, int of) { first[before + k] = (uint32_t)p | (uint32_t)(before + of) << 16; });
    if (lane == 63) *blocks = inc;
}

// Latency of one workgroup: everything but the lists themselves stays in LDS.  T = 8192: 17.9 us with clusters of twenty, 14.0
// with clusters of two; T = 2048: 7.5.
__global__ __launch_bounds__(SCREEN_SORT_THREADS) void k_screen_sort(ScreenFullParams f) {
    extern __shared__ __align__(16) char lds[];
    __shared__ int s_last[SORT_HEAD_BLOCKS], s_blocks;        // last head of a block; blocks of members
    __shared__ unsigned long long s_edge[SORT_HEAD_BLOCKS + 2];   // a bit where a cluster starts in the members' list
    __shared__ uint32_t s_first[SORT_MEMBER_BLOCKS];          // see SW_FIRST; as they come: the start of the cluster alone
    __shared__ int2 s_sum[2][SCREEN_SORT_THREADS / 64];
    const ScreenParams& p = f.s;
    const ScreenUnit U(p.T, p.nch, p.edge_cap);
    const int tid = threadIdx.x, T = p.T, Tp = (T + 63) & ~63;
    const uint32_t* hdr = reinterpret_cast<const uint32_t*>(p.area);
    const ScreenLists L = screen_full_lists(p, U);
    // The first workgroup sorts.  The others see to the unexplained candidates, if there are any: then the last one to be done sorts, as in
    // k_screen_chain.  (As a launch in front that left at once as a rule it took 2 to 4 us; looking at the counts here takes 0.6.  Full
    // selection, T=8192, d=4096 87.1 -> 83.9 us, greedy covering, T=2048, d=4096 50.8 -> 49.0.)
    __shared__ int s_state;
    __shared__ uint32_t s_pairs;
    uint32_t* cnt = reinterpret_cast<uint32_t*>(lds);         // members of a cluster; then the next free place in the list
    uint32_t* cl2 = cnt + Tp;                                 // two clusters per word; bit 15: an edge to an earlier token
    uint16_t* cl = reinterpret_cast<uint16_t*>(cl2);
    uint16_t* list = cl + Tp;
    auto take = [&] {
        for (int t = tid; t < Tp; t += SCREEN_SORT_THREADS) cnt[t] = 0u;
        if (tid < SORT_HEAD_BLOCKS + 2) s_edge[tid] = 0ull;
        for (int w = tid; w < Tp / 8; w += SCREEN_SORT_THREADS) reinterpret_cast<uint4*>(cl2)[w] = reinterpret_cast<const uint4*>(p.area + U.o_cl)[w];
    };
    if (blockIdx.x == 0) take();                              // (no candidate changes the clusters; the last wave has the header besides)
    if (tid >= SCREEN_SORT_THREADS - 64) {
        const ScreenCounts n = screen_counts(hdr);
        s_state = screen_state(p, n) | ((n.flags & SF_LOW) ? 16 : 0);
        s_pairs = n.pairs;
    }
    screen_barrier();
    const int state = __builtin_amdgcn_readfirstlane(s_state) & 15;
    const uint32_t pairs = s_pairs;
    if (state != UNIT_OPEN && blockIdx.x > 0) return;         // uniform
    if (state == UNIT_OPEN) {
        if (blockIdx.x > 0)
            screen_rest_tiles<SCREEN_SORT_THREADS, 1>(p, U, p.area, 0, 0, (s_state & 16) != 0, (int)blockIdx.x - 1, (int)gridDim.x - 1, f.ntile, f.lanes,
                                                   f.f32 != 0, lds);
        const int rest = (int)gridDim.x - 1;
        if (!screen_last(p.meta + META_WALK, blockIdx.x > 0 ? reinterpret_cast<uint32_t*>(p.area) : nullptr, (int)blockIdx.x - 1, rest, screen_groups(rest))) return;
        if (blockIdx.x > 0) take();
    }
    const uint32_t n_edge = state == UNIT_OPEN ? __hip_atomic_load(hdr + SU_EDGES, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
    const bool dense = state == UNIT_DENSE ||
                       (state == UNIT_OPEN && __hip_atomic_load(hdr + SU_DENSE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u);
    // (the greedy covering takes a token that only covered tokens cover: with edges it is resolved from the pair bits)
    if (dense || (f.greedy && n_edge) || (f.want_gamma && pairs > SCREEN_FULL_PAIRS * (uint32_t)T)) {
        if (tid == 0) { *f.gate = 1; L.work[SW_TILES] = 0; L.work[SW_TILES128] = 0; }
        return;
    }
    screen_barrier();
    for (int t = tid; t < T; t += SCREEN_SORT_THREADS) atomicAdd(&cnt[cl[t]], 1u);
    screen_barrier();
    if (n_edge) {
        for (uint32_t e = tid; e < n_edge; e += SCREEN_SORT_THREADS) {
            const uint32_t t = reinterpret_cast<const uint2*>(p.area + U.o_edge)[e].x & 0xFFFFu;
            atomicOr(&cl2[t >> 1], 0x8000u << (16 * (t & 1)));
        }
        screen_barrier();
    }
    const int chunk = (T + SCREEN_SORT_THREADS - 1) / SCREEN_SORT_THREADS;
    const int lo = min(T, tid * chunk), hi = min(T, lo + chunk);
    int n_mem = 0, n_head = 0, n_set = 0;
    for (int t = lo; t < hi; ++t) {
        const int n = (int)cnt[t], c = cl[t];
        n_mem += n > 1 ? n : 0;
        n_head += (c & 0x7FFF) == t;
        n_set += c == t;                                      // in the set: no earlier token within the threshold
    }
    int2 all;                                                 // (x: members and, from bit 16 on, heads; each at most 2^14)
    const int2 at = screen_scan(int2{n_mem | n_head << 16, n_set}, &all, s_sum[0]);
    const int mem = all.x & 0xFFFF, heads = all.x >> 16;
    // Blocks of 64 members as they come take a second tile for the cluster that goes over the edge in front; blocks of whole clusters
    // are about a tenth more, with one tile each, and take a chain of steps to find.  A tile takes its time however full it is, so the
    // second one costs nothing while all of them and those of the heads find a CU of their own: bf16, d = 4096, us, as they come and
    // whole: T = 2048, K = 400 49 and 54 (greedy covering), T = 4400, K = 400 56.9 and 59.1, T = 6000 70.9 and 64.6, T = 8192 84.5
    // and 77.8, T = 12000, K = 300 114.5 and 100.3.  Nor does it show beside the heads' tiles where clusters are small: T = 8192, K = 4000 186.4 and
    // 190.7.
    const bool whole = mem >= f.whole_from && heads * 8 <= mem;
    int o_mem = at.x & 0xFFFF, o_head = at.x >> 16, o_set = at.y;
    for (int t = lo; t < hi; ++t) {
        const int n = (int)cnt[t], c = cl[t];
        if (n > 1) {
            const bool large = whole ? n > 64 : (o_mem >> 6) != (o_mem + n - 1) >> 6;
            cnt[t] = SORT_PLACED | (large ? SORT_LARGE : 0u) | (uint32_t)o_mem;
            if (whole) atomicOr(&s_edge[o_mem >> 6], 1ull << (o_mem & 63));
            else for (int b = (o_mem + 63) >> 6; b * 64 < o_mem + n; ++b) s_first[b] = (uint32_t)o_mem;   // (the cluster that a block starts in)
            o_mem += n;
        }
        if ((c & 0x7FFF) == t) {
            if ((o_head & 63) == 63 || o_head == heads - 1) s_last[o_head >> 6] = t;
            L.head[o_head++] = t;
        }
        if (f.mask) f.mask[t] = c == t;
        if (c == t) { if (f.idx) f.idx[o_set] = t; ++o_set; }
    }
    if (tid == 0) {
        *f.gate = 0;
        *reinterpret_cast<int4*>(f.counts) = int4{all.y, all.y, 0, ADA_OK};
        if (f.ops) *f.ops = (unsigned long long)T * (unsigned long long)T;   // Table 6 / eq. (6)
    }
    if (!f.want_gamma) return;                                // uniform
    screen_barrier();
    for (int t = tid; t < T; t += SCREEN_SORT_THREADS) {
        uint32_t* c = &cnt[cl[t] & 0x7FFF];
        if (*c & SORT_PLACED) {
            const uint32_t v = atomicAdd(c, 1u);
            const int place = (int)(v & SORT_PLACE);
            list[place] = (uint16_t)t;
            if (!(v & SORT_LARGE)) L.member[place] = t;       // (the others below, in token order)
        }
    }
    if (whole && tid >= SCREEN_SORT_THREADS - 64) sort_blocks(s_edge, mem, s_first, &s_blocks);   // (one wave; the starts are known since the last barrier)
    screen_barrier();
    // tiles: a block of members each for the first threads, then a block of heads each
    const int blocks = whole ? s_blocks : (mem + 63) >> 6, head_blocks = (heads + 63) >> 6;
    auto first_of = [&](int b) { return whole ? s_first[b] : (uint32_t)(b * 64) | (s_first[b] >> 6) << 16; };
    int n = 0, n128 = 0;
    if (tid < blocks) n = tid - (int)(first_of(tid) >> 16) + 1;
    else if (tid < blocks + head_blocks) n = (s_last[tid - blocks] + 63) >> 6;
    if (tid <= blocks) L.work[SW_FIRST + tid] = tid < blocks ? (int)first_of(tid) : mem;
    if (tid < SORT_HEAD_BLOCKS / 2 && tid * 128 < heads) n128 = (s_last[min(2 * tid + 1, head_blocks - 1)] + 127) >> 7;
    int2 tiles;
    const int2 o = screen_scan(int2{n, n128}, &tiles, s_sum[1]);
    if (tid <= blocks + head_blocks) L.work[SW_PRE + tid] = o.x;   // (the last one has none: the total)
    if (tid <= SORT_HEAD_BLOCKS / 2) L.work[SW_PRE128 + tid] = o.y;
    if (tid == blocks) {
        const int nb = (T + 63) >> 6;
        const bool big = tiles.x - o.x >= f.big_tiles, most = (float)(tiles.x - o.x) > f.most_heads * (float)(nb * (nb + 1) / 2);
        L.work[SW_BLOCKS] = blocks;
        L.work[SW_HEADS] = heads;
        L.work[SW_TILES] = most ? 0 : big ? o.x : tiles.x;
        L.work[SW_TILES128] = big && !most ? tiles.y : 0;
        if (most) *f.gate = 1;
    }
    // a block meets the blocks before it only: clusters of several blocks go into token order
    // (sixteen lanes per cluster, a member's place is the number of smaller ones)
    for (int b = 1 + (tid >> 4); b < blocks; b += SCREEN_SORT_THREADS / 16) {
        if ((int)(first_of(b) >> 16) != b - 1) continue;       // (the second block of its cluster)
        const int st = whole ? (int)(s_first[b - 1] & 0xFFFFu) : (int)s_first[b], en = (int)(cnt[cl[list[st]] & 0x7FFF] & SORT_PLACE);
        for (int j = st + (tid & 15); j < en; j += 16) {
            const int v = list[j];
            int rank = 0;
#pragma unroll 8
            for (int i = st; i < en; ++i) rank += list[i] < v;
            L.member[st + rank] = v;
        }
    }
}

// Tile u -> the block it belongs to: the one that starts at or before it (256 threads; pre: n + 1 ascending words).
__device__ inline int screen_find(const int32_t* pre, int n, int u, int* s_found) {
    __syncthreads();                                          // (the tile before is done with *s_found)
    for (int i = threadIdx.x; i < n; i += 256)
        if (pre[i] <= u && u < pre[i + 1]) *s_found = i;
    __syncthreads();
    return *s_found;
}

// Bound by what a CU pulls out of the L2 (1 MB per 64 x 64 tile at d = 4096 in bf16).  XCD x takes a contiguous range of the
// heads' 128 x 128 tiles, then one of the 64 x 64 tiles.  T = 8192, d = 4096: 26 us at K = T / 20 (34 with two tiles per block
// of members), 150 us at K = T / 2, where 128 x 128 tiles replace 2600 small ones; the whole triangle takes 264 us.  DMA: whole 64-byte
// pieces of bf16 rows (see ada_gram_dma.hpp).
template <typename In, bool DMA>
__global__ __launch_bounds__(256) void k_screen_gram(ScreenParams sp, GramParams p) {
    extern __shared__ __align__(16) char lds[];
    __shared__ int s_found;
    const ScreenUnit U(sp.T, sp.nch, sp.edge_cap);
    const ScreenLists L = screen_full_lists(sp, U);
    const int total = L.work[SW_TILES], total128 = L.work[SW_TILES128], heads = L.work[SW_HEADS], blocks = L.work[SW_BLOCKS];
    const int per = (total + 7) >> 3, per128 = (total128 + 7) >> 3, xcd = (int)(blockIdx.x & 7);
    for (int slot = (int)(blockIdx.x >> 3); slot < per128 + per; slot += (int)(gridDim.x >> 3)) {
        if (slot < per128) {
            const int u = xcd * per128 + slot;
            if (u >= total128) continue;                      // uniform
            const int i = screen_find(L.work + SW_PRE128, SORT_HEAD_BLOCKS / 2, u, &s_found), s0 = (u - L.work[SW_PRE128 + i]) * 128;
            if constexpr (DMA) gram_tile_dma<64, true>(p, s0, i * 128, true, lds, L.head, heads);
            else gram_tile<In, 128, true>(p, nullptr, L.head, s0, i * 128, sp.T, heads, true, lds);
        } else {
            const int u = xcd * per + slot - per128;
            if (u >= total) break;                            // uniform
            const int i = screen_find(L.work + SW_PRE, blocks + ((heads + 63) >> 6), u, &s_found), k = u - L.work[SW_PRE + i];
            const bool m = i < blocks;
            int s0 = k * 64, t0 = (i - blocks) * 64, nS = sp.T, nT = heads;
            if (m) {
                const int32_t* at = L.work + SW_FIRST;
                const int sb = (at[i] >> 16) + k;
                s0 = at[sb] & 0xFFFF; nS = at[sb + 1] & 0xFFFF;
                t0 = at[i] & 0xFFFF; nT = at[i + 1] & 0xFFFF;
            }
            gram_tile<In, 64, true>(p, m ? L.member : nullptr, m ? L.member : L.head, s0, t0, nS, nT, true, lds);
        }
    }
}

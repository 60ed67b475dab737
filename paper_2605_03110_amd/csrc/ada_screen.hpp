// Screened selection: the sets of many layers from the GRAPH of near pairs.  Included by ada_kernels.hip after
// ada_fused.hpp.
//
// Definition 2.2 and Algorithm 1 only ask of a product whether |cos| reaches 1 - tau^2, and that question does not depend
// on the inherited set: the pairs of tokens within the threshold of each other are a property of a layer's X alone.  So
// they are found for all layers of a call at once, where the chip is full, and what stays sequential from layer to layer
// is a walk over that graph by one workgroup.  Finding them does not take T^2 / 2 full products either:
//
//   sketch  n1 of the d columns (whole groups of 64, spread evenly over the row) of every row, scaled to unit length and
//           rounded to 8-bit floats.  For a pair (s, t) with the cosine c1 of its two sketches,
//               |cos(s,t)| <= rho_s rho_t |c1| + sqrt(1 - rho_s^2) sqrt(1 - rho_t^2)        (Cauchy-Schwarz on the rest)
//           where rho^2 is the share of a row's squared norm that the sketch holds.  A pair whose sketch product stays
//           below kappa is therefore within the threshold ONLY IF a row holds unusually little in the sketch; with every
//           rho^2 at least f2 it is certainly not: the bound over all such rows is 1 - (1 - kappa') f2, kappa' = kappa plus
//           the worst rounding of both sketches (see ScreenPlan).  What is left are the CANDIDATE pairs.
//   pairs   all sketch products on MFMA; every token keeps its earliest candidate, its PIVOT.
//   exact   one full product per token, with its pivot, in the precision of the other paths, and every row's norm: one
//           pass over X.  A token close to its pivot (angle at most 0.45 of the threshold's) joins the pivot's CLUSTER:
//           acos |cos| is a metric, so all members of a cluster are within the threshold of each other.
//   rest    candidate pairs that no cluster explains are multiplied out one by one and become EDGES (a pair
//           and its cosine).  Whether there are
//           any is a matter of counting: with every rho^2 >= f2 all pairs inside clusters are candidates, so if there are
//           exactly as many candidates as pairs inside clusters there is nothing else.
//   chain   one workgroup per sequence walks through the layers: Definition 2.2 at layer 0, Algorithm 1 afterwards, on the
//           clusters and edges alone.  One launch with `rest`, whose workgroups leave at once as a rule.
// Nothing here is approximate: a pair is decided by its full product, by the metric or by the bound, with margins
// (1e-4 on |cos| and more) far above the rounding of any of them.  Where the data do not cooperate -- so many pairs near the
// threshold that listing them is no saving -- a layer is marked DENSE and the launch behind the chain runs it and the
// layers after it on the tiles of the other path.
//
// Measured (bf16, tau = 0.1): see the kernels below.
#pragma once

constexpr int SCREEN_MAX_LAYERS = 64;                         // layers per launch (their pointers travel as arguments)
constexpr int SCREEN_TILE_PAIRS = 256;                        // unexplained candidates a 128 x 128 tile may hold before its layer is dense
// Unexplained candidates per token from which on a layer is dense without looking at them: listing one takes two rows out of the
// L2 (16 KB at d = 4096, 1.1 ns of the chip), a step on the tiles 27 us at T = 2048, 150 us at T = 8192.  All of them may turn
// out to be edges, and the walk goes along edges at about 1.5 us per thousand: 28 layers of T=2048, d=4096 with 2.2 unexplained
// candidates per token take 673 us on the graph and 1270 with one launch per layer.  A launch of many layers has room for
// fewer edges, and then that is the line; screen_edges what it always has.
constexpr int SCREEN_OPEN = 4;
constexpr int screen_edges(int T) { return (T / 2 + 65) / 2 * 2; }
constexpr int CHAIN_LDS = 160 * 1024 - 2048;                  // what the walk may use of a CU's LDS
// Sketches are stored as 8-bit floats of scale x (unit vector), the products multiplied by a power of two so that the
// accumulators hold 2 c / kappa: scale^2 = 2 / (kappa 2^SCREEN_EXP), below the formats' largest 448 for every kappa >= 0.3.
constexpr int SCREEN_EXP = -14;

// header of a unit (one layer of one sequence); zeroed by the sketch launch
enum { SU_EDGES = 3, SU_DENSE = 4, SU_CAND = 32, SU_PART = SU_CAND + 8 * 32, SU_WORDS = SU_PART + 8 * 32 };
// What every workgroup of the pair and exact passes adds to is kept once per XCD, a cache line each, from words SU_CAND and
// SU_PART on (lines of their own: the exact pass reads the candidates while it counts the pairs): one address takes an atomic every 25 ns from the whole chip, which was most of these passes where one unit has all the
// workgroups (T = 8192, d = 4096: pairs 18.6 -> 13.6 us, exact 35.4 -> 20.7 us; T = 2048: 5.6 -> 5.2 and 11.8 -> 9.0).
enum { SU_PAIRS = 0, SU_FLAGS = 1, SU_DONE = 2 /* sign-offs of the unit's workgroups, see screen_last */ };
enum { SF_LOW = 1, SF_MESH = 2 };                             // SU_FLAGS: a row below f2; a pivot that has a pivot itself

struct ScreenCounts { uint32_t cand, pairs, flags; };
__device__ inline ScreenCounts screen_counts(const uint32_t* hdr) {
    ScreenCounts n = {0u, 0u, 0u};
#pragma unroll
    for (int x = 0; x < 8; ++x) {
        n.cand += hdr[SU_CAND + x * 32];
        n.pairs += hdr[SU_PART + x * 32 + SU_PAIRS];
        n.flags |= hdr[SU_PART + x * 32 + SU_FLAGS];
    }
    return n;
}

// How a problem is screened (host): columns of the sketch and the constants of the bound.
struct ScreenPlan {
    int nch;            // column groups of 64 in the sketch
    float kappa;        // candidate: sketch product at least this (before rounding allowance)
    float f2;           // rows must hold at least this share of their squared norm in the sketch
    float safe;         // 1 - tau^2 minus the margin
    float cos_tight;    // cosine of 0.45 of the threshold's angle
};
constexpr double SCREEN_EPS = 0.13;                           // 2 d + d^2 for a rounding of d = 2^-4 on each side (0.1289), and what underflows

// nch: the smallest sketch for which ordinary rows pass.  kappa is where two unrelated rows stop to occur among all pairs of
// a long sequence (the cosine of two independent directions in n dimensions exceeds k with probability about
// (1 - k^2)^((n-1)/2); 3e-10 here), f2 follows from it, and n1 is taken where the share of the norm that n1 of d columns
// of independent entries hold lies above f2 with 4.3 standard deviations (Wilson-Hilferty).  More than half of the
// columns, or a threshold no bound reaches: not screened.
// Small thresholds: two members of a cluster are not multiplied, each is at most 0.45 of the threshold's angle from the
// pivot, so their cosine lies above the threshold by cos(0.9 acos(thr)) - thr, about 0.19 tau^2.  A rounding of r on each of
// the two cosines with the pivot comes off that four-fold (angles add: (a + b)^2 / 2 with a = b and a^2 = 2 (1 - cos)).  r:
// lane sums of d / 64 products (up to 64 in short rows) and their reduction, of the product and, halved twice, of two
// squared norms.  What is left has to be 1e-4, as at the other decisions: tau >= 0.027 up to d = 4096.
inline bool screen_plan(int d, float tau, ScreenPlan* out) {
    const double thr = 1.0 - (double)tau * (double)tau, safe = thr - 2e-4;
    const int nk = (d + 63) / 64;
    if (d < 64) return false;
    const double rounding = 2.0 * ((d > 4096 ? d / 64.0 : 64.0) + 16.0) / (1 << 24);
    if (cos(0.9 * acos(thr)) - thr < 1e-4 + 4.0 * rounding) return false;
    for (int nch = 1; nch <= nk; ++nch) {
        const int n = 64 * nch, ne = n < d ? n : d;
        double k = sqrt(1.0 - exp(-44.0 / (ne - 1)));
        if (k < 0.3) k = 0.3;
        const double kap = k + SCREEN_EPS;
        double f2 = 0.0;
        if (nch == nk) {                                       // the sketch is the row: the product itself, rounded
            if (nch > 4 || kap > safe - 5e-3) return false;
        } else {
            if (kap > 0.93) continue;
            f2 = (1.0 - safe) / (1.0 - kap);
            const double wh = 1.0 - 2.0 / (9.0 * n) - 4.3 * sqrt(2.0 / (9.0 * n));
            if ((double)n / d * wh * wh * wh < f2) continue;
            if (n > 512 && 2 * n > d) return false;
        }
        out->nch = nch;
        out->kappa = (float)k;
        out->f2 = (float)f2;
        out->safe = (float)safe;
        out->cos_tight = (float)cos(0.45 * acos(thr));
        return true;
    }
    return false;
}

// Memory of a unit inside the workspace's screen area, in bytes from the unit's start.  Sketches lie in the order in which
// a wave loads them as matrix operands: blocks of 32 rows, in a block column group after column group, a group as two
// runs of 64 lanes x 16 bytes (lane l: row l % 32, columns 32 (l / 32) + 16 run .. + 15), so that every operand load is one
// kilobyte without gaps.
// edge_cap: places for edges, as many as the launch has room for (even).
struct ScreenUnit {
    int o_piv, o_size, o_rho, o_cl, o_mask, o_edge, o_z, edge_cap;
    long long bytes;
    __host__ __device__ ScreenUnit(int T, int nch, int edges) {
        const long long t4 = (long long)align_up((size_t)T * 4, 256);
        edge_cap = edges;
        long long o = SU_WORDS * 4;
        o_piv = (int)o; o += t4;
        o_size = (int)o; o += t4;
        o_rho = (int)o; o += t4;
        o_cl = (int)o; o += (long long)align_up((size_t)T * 2, 256);
        o_mask = (int)o; o += (long long)align_up((size_t)((T + 63) / 64) * 16, 256);   // the set, and the one inherited by a launch's first layer
        o_edge = (int)o; o += (long long)align_up((size_t)edge_cap * 8, 256);
        o_z = (int)o; o += (long long)((T + 31) / 32) * nch * 2048;
        bytes = (long long)align_up((size_t)o, 256);
    }
};

struct ScreenParams {
    long long ld;
    int T, d;
    int G, L;                  // sequences (or heads), layers of this launch
    long long x_gs;            // bytes between sequences' X
    char* area;                // sequence 0's screen area; the others area_gs bytes apart
    long long area_gs;
    int32_t* meta;             // sequence 0's scalars (likewise area_gs apart)
    int first;                 // layer number of the launch's first layer
    int nch, nk;
    float scale, kap1;         // of the stored sketches; kappa with the rounding allowance
    float f2, safe, thr, cos_tight;
    uint32_t open;             // unexplained candidates of a unit above which it is dense
    int edge_cap;              // see ScreenUnit
    int count_pairs;           // the exact pass counts the pairs inside clusters (else k_screen_rest does)
    float* gamma;              // one unit: largest |cos| of the pairs multiplied out (bits under an integer max), or NULL
    float* inv_norm;           // one unit: inverse norms of the rows, or NULL
    const void* X[SCREEN_MAX_LAYERS];
};

__device__ inline char* screen_unit(const ScreenParams& p, const ScreenUnit& U, int unit, int* layer, int* group) {
    const int l = unit / p.G, g = unit - l * p.G;
    *layer = l;
    *group = g;
    return p.area + (long long)g * p.area_gs + (long long)l * U.bytes;
}

template <typename In>
__device__ inline const In* screen_x(const ScreenParams& p, int layer, int group) {
    return reinterpret_cast<const In*>(reinterpret_cast<const char*>(p.X[layer]) + (long long)group * p.x_gs);
}

// Eight consecutive elements from column e0 on, as floats; columns at or beyond d are zero.  The load is pulled back
// into the row and what it repeats is cleared, so rows of any length and alignment are read in whole pieces (d >= 8).
template <typename In> __device__ inline void screen_load8(const In* row, int e0, int d, float (&v)[8]);
template <> __device__ inline void screen_load8<uint16_t>(const uint16_t* row, int e0, int d, float (&v)[8]) {
    const int e = min(e0, d - 8), cut = e0 - e;
    const u32x4 r = *reinterpret_cast<const u32x4_any*>(row + e);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = 2 * i >= cut ? __uint_as_float(r[i] << 16) : 0.f;
        v[2 * i + 1] = 2 * i + 1 >= cut ? __uint_as_float(r[i] & 0xFFFF0000u) : 0.f;
    }
}
template <> __device__ inline void screen_load8<float>(const float* row, int e0, int d, float (&v)[8]) {
    const int e = min(e0, d - 8), cut = e0 - e;
    const u32x4 a = *reinterpret_cast<const u32x4_any*>(row + e), b = *reinterpret_cast<const u32x4_any*>(row + e + 4);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[i] = i >= cut ? __uint_as_float(a[i]) : 0.f;
        v[4 + i] = 4 + i >= cut ? __uint_as_float(b[i]) : 0.f;
    }
}

// All waves' LDS operations done, and everybody here.  (A fenced barrier would also wait for
// the loads and stores in flight to memory, a microsecond or two in which a finished workgroup keeps its place.)
__device__ inline void screen_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// ------------------------------------------------------------------------------------------------
// k_screen_sketch: eight lanes per row, eight columns per lane and column group.  Reads n1 / d of X, one cache line (two
// for fp32) per row and group; all that a lane needs is requested before the first of it is used.  NCH: column groups, or 0:
// more than four (the first four requested together).  R: rows per lane.  Four where a row is one line and there are many of them,
// or the launch is bound by the dispatch of its workgroups (128 units of T=2048, d=256: 20.4 us with one row, 13.0 with four).
constexpr int SKETCH_ROWS = 32;                               // rows per workgroup and pass
template <typename In, int NCH, int R>
__global__ __launch_bounds__(256) void k_screen_sketch(ScreenParams p, int row_blocks) {
    const ScreenUnit U(p.T, p.nch, p.edge_cap);
    const int unit = blockIdx.x / row_blocks, rb = blockIdx.x - unit * row_blocks;
    int layer, group;
    char* base = screen_unit(p, U, unit, &layer, &group);
    const In* X = screen_x<In>(p, layer, group);
    if (rb == 0) {
        for (int i = threadIdx.x; i < SU_WORDS; i += 256) reinterpret_cast<uint32_t*>(base)[i] = 0u;
        // words of the call (not of the unit): layers done so far; the last launch's queue is left at zero by itself
        if (layer == 0 && p.first == 0 && threadIdx.x == 0)
            reinterpret_cast<int32_t*>(reinterpret_cast<char*>(p.meta) + (long long)group * p.area_gs)[META_PROGRESS] = 0;
    }
    constexpr int KEEP = NCH > 0 ? NCH : 4;
    const int nch = NCH > 0 ? NCH : p.nch;
    const int lane = threadIdx.x & 63, c8 = lane & 7;
    const int t0 = rb * SKETCH_ROWS * R + (threadIdx.x >> 6) * 8 + (lane >> 3);
    auto row = [&](int k) { return X + (size_t)min(t0 + k * SKETCH_ROWS, p.T - 1) * (size_t)p.ld; };
    auto col = [&](int j) { return (int)((unsigned)j * (unsigned)p.nk / (unsigned)nch) * 64 + c8 * 8; };
    float v[R][KEEP][8];
#pragma unroll
    for (int k = 0; k < R; ++k)
#pragma unroll
        for (int j = 0; j < KEEP; ++j) screen_load8<In>(row(k), col(j), p.d, v[k][j]);
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int t = t0 + k * SKETCH_ROWS;
        float ss = 0.f;
#pragma unroll
        for (int j = 0; j < KEEP; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i) ss = fmaf(v[k][j][i], v[k][j][i], ss);
        for (int j = KEEP; j < nch; ++j) {
            float x[8];
            screen_load8<In>(row(k), col(j), p.d, x);
#pragma unroll
            for (int i = 0; i < 8; ++i) ss = fmaf(x[i], x[i], ss);
        }
        ss += __shfl_xor(ss, 1, 64);
        ss += __shfl_xor(ss, 2, 64);
        ss += __shfl_xor(ss, 4, 64);
        const float sc = ss > 0.f ? p.scale / sqrtf(ss) : 0.f;
        if (t >= p.T) return;                                 // (and so are the lane's other rows)
        uint8_t* z = reinterpret_cast<uint8_t*>(base + U.o_z) + (size_t)(t >> 5) * (size_t)(2048 * nch) +
                     ((c8 >> 1) & 1) * 1024 + ((c8 >> 2) * 32 + (t & 31)) * 16 + (c8 & 1) * 8;
        auto put = [&](int j, const float (&x)[8]) {
            int lo = 0, hi = 0;
            lo = __builtin_amdgcn_cvt_pk_fp8_f32(x[0] * sc, x[1] * sc, lo, false);
            lo = __builtin_amdgcn_cvt_pk_fp8_f32(x[2] * sc, x[3] * sc, lo, true);
            hi = __builtin_amdgcn_cvt_pk_fp8_f32(x[4] * sc, x[5] * sc, hi, false);
            hi = __builtin_amdgcn_cvt_pk_fp8_f32(x[6] * sc, x[7] * sc, hi, true);
            *reinterpret_cast<int2*>(z + j * 2048) = int2{lo, hi};
        };
#pragma unroll
        for (int j = 0; j < KEEP; ++j) put(j, v[k][j]);
        for (int j = KEEP; j < nch; ++j) {
            float x[8];
            screen_load8<In>(row(k), col(j), p.d, x);
            put(j, x);
        }
        if (c8 == 0) {
            reinterpret_cast<float*>(base + U.o_rho)[t] = ss;
            reinterpret_cast<int32_t*>(base + U.o_piv)[t] = t;
            reinterpret_cast<int32_t*>(base + U.o_size)[t] = 0;
            if (p.gamma) p.gamma[t] = 0.f;
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Sketch products.  The order of an operand's columns does not matter as long as both sides use the same one.
typedef int i32x8 __attribute__((ext_vector_type(8)));
__device__ inline i32x8 screen_operand(const u32x4* z) {      // this lane's 32 bytes of a (row block, column group)
    const u32x4 a = z[0], b = z[64];
    return i32x8{(int)a[0], (int)a[1], (int)a[2], (int)a[3], (int)b[0], (int)b[1], (int)b[2], (int)b[3]};
}
__device__ inline void screen_mma(f32x16& acc, const i32x8& a, const i32x8& b) {
    // (formats 0: e4m3 on both sides; block scale 127 + n: 2^n)
    constexpr int scale = (127 + SCREEN_EXP / 2) * 0x01010101;
    acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 0, 0, 0, scale, 0, scale);
}

// lower-triangular block number -> blocks 0 <= sb <= tb
__device__ inline void screen_blocks(int tile, int* sb, int* tb) {
    int n = (int)((sqrtf(8.f * (float)tile + 1.f) - 1.f) * 0.5f);
    while ((n + 1) * (n + 2) / 2 <= tile) ++n;
    while (n * (n + 1) / 2 > tile) --n;
    *tb = n;
    *sb = tile - n * (n + 1) / 2;
}

// The candidates of a 32 x 32 block: sketches and block scales are such that an accumulator holds 2 c / kappa, so a candidate
// is an accumulator whose exponent has its top bit set (bit 30).  One instruction per product: it shifts that bit and the
// sign in from the right; the caller masks the signs away (SCREEN_BITS).  Register i lands in bit 30 - 2 i and holds a row that
// grows with i, so the highest bit is the earliest row.
constexpr uint32_t SCREEN_BITS = 0x55555555u;
__device__ inline uint32_t screen_bits(const f32x16& acc) {
    uint32_t bits = 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(acc[i]), 30u);
    return bits;
}
__device__ inline int screen_row(int i) { return (i & 3) + 8 * ((i >> 2) & 3); }   // row of register i (lanes of the first half)
__device__ inline uint32_t screen_first(uint32_t bits) {      // position of the highest bit from the left; all ones if there is none
    uint32_t r;
    asm("v_ffbh_u32 %0, %1" : "=v"(r) : "v"(bits));
    return r;
}

// Work items of a unit: strips of 256 tokens, each against its earlier tokens in pieces.  A piece is 256 x `wide` tokens, or
// 256 / `cut` of them: long pieces spend less of their time on starting up (a piece of 256 took about half of it for
// that), short ones are needed to fill the chip.  Two workgroups per CU fill it: halved pieces up to four per CU cost a layer
// loop of 12 x T=2048, d=768 50.8 us instead of 48.7, 2 x T=4096, d=512 36.0 instead of 34.0.  With one column group a piece has a
// third of the products: 128 x T=2048, d=256 29.3 us in pieces of 256, 26.5 of 512, 27.0 of 1024; calls in pieces of 256 and of 512, by their tiles: T=2048,
// 1152 42.5 and 42.3, 2016 52.9 and 52.3, 2304 55.8 and 54.2, 4608 81.6 and 77.6, T=8192, 2112 40.2 and 38.9, 4224 62.6 and 60.1.  Strips come in groups of
// `wide` with the same number of pieces.
struct PairItems {
    int wide, cut, per_unit;
    __host__ __device__ PairItems(int T, int units, int nch) {
        const int nb = (T + 255) / 256;
        const long long tiles = (long long)nb * (nb + 1) / 2 * units;
        wide = tiles >= 12288 ? 4 : tiles >= (nch == 1 ? 2048 : 6144) ? 2 : 1;
        cut = tiles >= 512 ? 1 : tiles >= 256 ? 2 : 4;
        const int q = (nb + wide - 1) / wide;
        per_unit = wide * (q * (q + 1) / 2) * cut;
    }
    // item -> strip, first block of 32 earlier tokens, number of blocks (clipped by the caller)
    __device__ void get(int i, int* tb, int* s_lo, int* sblk) const {
        if (cut > 1) {
            int a, b;
            screen_blocks(i / cut, &a, &b);
            *tb = b;
            *sblk = 8 / cut;
            *s_lo = a * 8 + (i % cut) * (8 / cut);
            return;
        }
        int a, q;
        screen_blocks(i / wide, &a, &q);                      // group q: wide (q + 1) items from wide q (q + 1) / 2 on
        const int r = i - wide * (q * (q + 1) / 2);
        *tb = wide * q + r / (q + 1);
        *sblk = 8 * wide;
        *s_lo = (r % (q + 1)) * 8 * wide;
    }
};

// k_screen_pairs: every token's earliest candidate, and how many candidate pairs there are.  A workgroup holds 256 tokens
// and walks over blocks of 32 earlier tokens; a wave keeps TB blocks of tokens in registers and reads the earlier tokens'
// sketches once for all of them, a block ahead.  Waves that read the same blocks do so at about the same time, so they come
// from the L1; there is nothing to stage and no barrier.  TB = 4: two waves share the tokens, and the other two take the
// second half of the earlier tokens; TB = 2: four waves share the tokens.  The work of one unit is dealt to one XCD
// (workgroup b runs on XCD b % 8), so that its sketches are read by one L2.
// Bound by the matrix cores at the clock that they leave: 32 x T=8192 with three column groups keep the 8-bit MFMA busy for 66% of
// 304 thousand cycles, 157 us at 1.94 GHz (the exact pass beside it runs at 2.28): 2.7 PFLOP/s.
// Calls, us, with two blocks per wave, two instructions per product and two sets of operands (before) and now: 4 x 8 x T=8192,
// d=4096 619 -> 596, 128 x T=2048, d=256 105 -> 99, 12 x T=2048, d=768 46.7 -> 45.3.  Slower: sketches by way of LDS (607), two
// waves per SIMD with the operands a whole step ahead (616).
// NCH: column groups of the sketch (1 .. 4), or 0: any number, both operands read as they are used.
// (the second launch bound keeps the accumulators in ordinary registers: the epilogue reads each of them once)
constexpr int screen_pair_waves(int nch, int tb) { return nch == 1 ? 5 : nch == 2 && tb == 4 ? 4 : 3; }
template <int NCH, int TB>
__global__ __launch_bounds__(256, screen_pair_waves(NCH, TB)) void k_screen_pairs(ScreenParams p, PairItems it, int total) {
    constexpr int HELD = NCH > 0 ? NCH : 1, ACC = NCH > 0 ? 2 : TB;
    __shared__ int s_cand;
    const int per = (total + 7) >> 3;
    const int w = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (w >= total || (int)(blockIdx.x >> 3) >= per) return;
    const ScreenUnit U(p.T, p.nch, p.edge_cap);
    const int unit = w / it.per_unit;
    int layer, group, tb, s_lo, sblk;
    char* base = screen_unit(p, U, unit, &layer, &group);
    it.get(w - unit * it.per_unit, &tb, &s_lo, &sblk);
    if (threadIdx.x == 0) s_cand = 0;
    screen_barrier();
    const int T = p.T, nch = NCH > 0 ? NCH : p.nch, nblk = (T + 31) >> 5;
    const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int tb0 = tb * 8 + (TB == 4 ? (wave & 1) * 4 : wave * 2);           // this wave's first row block
    const int mid = TB == 4 ? s_lo + (sblk >> 1) : s_lo;
    int s = TB == 4 && wave >> 1 ? mid : s_lo;
    const int s_hi = min(TB == 4 && !(wave >> 1) ? mid : s_lo + sblk, min(tb0 + TB, nblk));
    const char* zb = base + U.o_z;                            // a (block, group) is 2 KB
    const uint32_t l16 = (uint32_t)lane * 16u;
    auto operand = [&](int n) { return screen_operand(reinterpret_cast<const u32x4*>(zb + (size_t)n * 2048 + l16)); };
    if (tb0 < nblk && s < s_hi) {
        i32x8 fb[TB][HELD], fa[HELD];
        uint32_t first[TB];                                   // block and bit of the earliest candidate: 32 s + position
        int cand = 0;
        auto rd = [&](i32x8 (&f)[HELD], int blk) {
            if constexpr (NCH > 0) {
#pragma unroll
                for (int j = 0; j < NCH; ++j) f[j] = operand(blk * NCH + j);
            }
        };
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            first[b] = 0xFFFFFFFFu;
            rd(fb[b], min(tb0 + b, nblk - 1));
        }
        rd(fa, s);
        if constexpr (NCH > 0) {
            if ((tb0 + TB) * 32 > T) {                        // (see block)
#pragma unroll
                for (int b = 0; b < TB; ++b)
                    if ((tb0 + b) * 32 + l32 >= T) {
#pragma unroll
                        for (int j = 0; j < NCH; ++j) fb[b][j] = i32x8{0, 0, 0, 0, 0, 0, 0, 0};
                    }
            }
        }
        uint32_t earlier = 0u;                                // on the diagonal: rows before this lane's
#pragma unroll
        for (int i = 0; i < 16; ++i) earlier |= 4 * half + screen_row(i) < l32 ? 0x40000000u >> (2 * i) : 0u;
        auto block = [&](int s, bool diag) {
#pragma unroll
            for (int b0 = 0; b0 < TB; b0 += ACC) {
                f32x16 acc[ACC];
#pragma unroll
                for (int b = 0; b < ACC; ++b)
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[b][i] = 0.f;
                if constexpr (NCH > 0) {
#pragma unroll
                    for (int j = 0; j < NCH; ++j)
#pragma unroll
                        for (int b = 0; b < ACC; ++b) screen_mma(acc[b], fa[j], fb[b0 + b][j]);
                    if (b0 + ACC == TB) {                     // the next block's operands, where the last product has taken this one's
                        __builtin_amdgcn_sched_barrier(0);
                        rd(fa, min(s + 1, s_hi - 1));
                        __builtin_amdgcn_sched_barrier(0);
                    }
                } else {
                    for (int j = 0; j < nch; ++j) {
                        const i32x8 a = operand(s * nch + j);
#pragma unroll
                        for (int b = 0; b < ACC; ++b) screen_mma(acc[b], a, operand(min(tb0 + b, nblk - 1) * nch + j));
                    }
                }
#pragma unroll
                for (int b = 0; b < ACC; ++b) {
                    uint32_t v = screen_bits(acc[b]) & (!diag || s < tb0 + b0 + b ? SCREEN_BITS : s == tb0 + b0 + b ? earlier : 0u);
                    // Tokens that do not exist have no candidates.  Their operands are zero, and so are their products with rows that were
                    // written; the last block's other rows, which only the diagonal meets, hold anything, and 0 x NaN is NaN.
                    if ((NCH == 0 || diag) && (tb0 + b0 + b) * 32 + l32 >= T) v = 0u;
                    cand += __popc(v);
                    first[b0 + b] = min(first[b0 + b], screen_first(v) | (uint32_t)s << 5);
                }
            }
        };
        for (; s < min(s_hi, tb0); ++s) block(s, false);     // whole blocks of earlier tokens
        for (; s < s_hi; ++s) block(s, true);
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const int t = (tb0 + b) * 32 + l32;
            const int i = (int)(first[b] & 31u) >> 1, row = (int)(first[b] >> 5) * 32 + 4 * half + screen_row(i);
            const int mine = first[b] == 0xFFFFFFFFu ? INT_MAX : row, q = min(mine, __shfl_xor(mine, 32, 64));
            if (half == 0 && t < T && q != INT_MAX) atomicMin(reinterpret_cast<int32_t*>(base + U.o_piv) + t, q);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) cand += __shfl_xor(cand, o, 64);
        if (lane == 0 && cand) atomicAdd(&s_cand, cand);
    }
    screen_barrier();
    if (threadIdx.x == 0 && s_cand)
        atomicAdd(reinterpret_cast<uint32_t*>(base) + SU_CAND + (blockIdx.x & 7) * 32, (uint32_t)s_cand);
}

// Sketch products of a 128 x 128 tile: four waves in a 2 x 2 grid of 64 x 64, 32 NB tokens (blocks b0 ..) at a time.
struct ScreenTile { int s0, t0; bool any; };                  // this wave's first rows; any: some s < t
__device__ inline ScreenTile screen_tile(int T, int sb, int tb, int wave) {
    const int s0 = sb * 128 + (wave >> 1) * 64, t0 = tb * 128 + (wave & 1) * 64;
    return {s0, t0, s0 <= t0 && t0 < T};                      // (not any: above the diagonal, or past the end)
}
template <int NB>
__device__ inline void screen_tile_products(const char* z, int T, int nch, const ScreenTile& me, int b0, f32x16 (&acc)[2][NB]) {
    const u32x4* Z = reinterpret_cast<const u32x4*>(z) + (threadIdx.x & 63);
    const int last = (T - 1) >> 5;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;
    for (int j = 0; j < nch; ++j) {
        i32x8 fa[2], fb[NB];
#pragma unroll
        for (int a = 0; a < 2; ++a) fa[a] = screen_operand(Z + (size_t)(min((me.s0 >> 5) + a, last) * nch + j) * 128);
#pragma unroll
        for (int b = 0; b < NB; ++b) fb[b] = screen_operand(Z + (size_t)(min((me.t0 >> 5) + b0 + b, last) * nch + j) * 128);
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < NB; ++b) screen_mma(acc[a][b], fa[a], fb[b]);
    }
}

// ------------------------------------------------------------------------------------------------
// Products of whole rows, piece by piece (see fetch_piece).
template <typename In> __device__ inline float screen_dot(u32x4 a, u32x4 b, float s);
template <> __device__ inline float screen_dot<float>(u32x4 a, u32x4 b, float s) {
#pragma unroll
    for (int i = 0; i < 4; ++i) s = fmaf(__uint_as_float(a[i]), __uint_as_float(b[i]), s);
    return s;
}
template <> __device__ inline float screen_dot<uint16_t>(u32x4 a, u32x4 b, float s) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const uint32_t a0 = a[0], a1 = a[1], a2 = a[2], a3 = a[3], b0 = b[0], b1 = b[1], b2 = b[2], b3 = b[3];
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a0), __builtin_bit_cast(bf16x2, b0), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a1), __builtin_bit_cast(bf16x2, b1), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a2), __builtin_bit_cast(bf16x2, b2), s, false);
    s = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a3), __builtin_bit_cast(bf16x2, b3), s, false);
    return s;
}

// <x, y>, <x, x> and <y, y> (TWO; else <x, x> alone) by LPR neighbouring lanes (li: this lane's place among them); every lane gets the sums.
// UN pieces of each row are requested before the first is used (four; eight leave fewer waves room: 465 us instead of 444 at
// 32 units of T = 8192, d = 4096).  STREAM: x is read once and not kept in the caches.  WHOLE: a row is so many times UN pieces of all
// lanes, so no piece is pulled back into it, cut or left out.
template <typename In, int LPR, bool STREAM = false, int UN = 4, bool WHOLE = false, bool TWO = true>
__device__ inline void screen_products(const In* x, const In* y, int d, int li, float* xy, float* xx, float* yy) {
    constexpr int EPP = 16 / (int)sizeof(In);
    const int np = (d + EPP - 1) / EPP;
    float sxy = 0.f, sxx = 0.f, syy = 0.f;
    for (int p0 = li; p0 < np; p0 += LPR * UN) {
        u32x4 a[UN], b[UN];
        auto from = [&](int u) { return WHOLE ? (p0 + u * LPR) * EPP : min(min(p0 + u * LPR, np - 1) * EPP, d - EPP); };
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const auto* piece = reinterpret_cast<const u32x4_any*>(x + from(u));
            if constexpr (STREAM) a[u] = __builtin_nontemporal_load(piece);
            else a[u] = *piece;
        }
        if constexpr (TWO) {
#pragma unroll
            for (int u = 0; u < UN; ++u) b[u] = *reinterpret_cast<const u32x4_any*>(y + from(u));
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int pc = p0 + u * LPR;
            if (WHOLE || pc < np) {
                const int cut = WHOLE ? 0 : pc * EPP - min(pc * EPP, d - EPP);
                const u32x4 va = cut > 0 ? clear_head<In>(a[u], cut) : a[u];
                sxx = screen_dot<In>(va, va, sxx);
                if constexpr (TWO) {
                    sxy = screen_dot<In>(va, b[u], sxy);
                    const u32x4 vb = cut > 0 ? clear_head<In>(b[u], cut) : b[u];
                    syy = screen_dot<In>(vb, vb, syy);
                }
            }
        }
    }
#pragma unroll
    for (int o = LPR / 2; o > 0; o >>= 1) {
        sxx += __shfl_xor(sxx, o, 64);
        if constexpr (TWO) {
            sxy += __shfl_xor(sxy, o, 64);
            syy += __shfl_xor(syy, o, 64);
        }
    }
    *xy = sxy;
    *xx = sxx;
    *yy = syy;
}

__device__ inline float screen_cos(float xy, float xx, float yy) {
    const float ix = xx > 0.f ? 1.0f / sqrtf(xx) : 0.f, iy = yy > 0.f ? 1.0f / sqrtf(yy) : 0.f;
    return (fabsf(xy) * ix) * iy;                             // a zero row normalises to zero: all its cosines are 0
}

// (screen_state has to agree: a quarter of the pairs is more than SCREEN_OPEN per token.  The full selection needs the norms
// in any case.  Nobody writes the counts while they are read here, so scalar loads will do; for short rows and sequences the
// wait for them is not worth the pass they may save: 0.5 of 8 us at 12 x 512 x 768 in fp32, 1 of 34 us at 128 x 2048 x 256.)
__device__ inline bool screen_crowded(const ScreenParams& p, const char* unit) {
    static_assert(1024 / 8 > SCREEN_OPEN, "crowded units are dense");
    if (p.T < 1024 || p.inv_norm) return false;
    const auto* cand = (const __attribute__((address_space(4))) uint32_t*)(unit) + SU_CAND;
    uint32_t n = 0u;
#pragma unroll
    for (int x = 0; x < 8; ++x) n += cand[x * 32];
    return n > (uint32_t)p.T * (uint32_t)p.T / 8u;
}

// k_screen_exact: norm of every row, product with its pivot, cluster.  HBM: X once.  Every XCD takes a contiguous range of
// the rows of all units, so that a unit's pivots (a few hundred rows, a few MB) are read into one L2 and not into eight.
// What a row needs besides X (pivot, sketch norm, the pivot's own pivot) is requested for all of a lane group's rows at
// once, a row's sums go to a lane of their own, and what follows from them is done once for all of them; no wave waits for its
// stores.  Instructions bind short rows and cost long ones waves in flight: 28 x T=2048, d=4096 86.8 -> 83.7 us, 32 x T=8192 389 -> 380,
// 16 heads x 256, 8 layers 34.3 -> 28.0 (before: pieces clamped, cut and left out one by one, every row's divisions, fenced barriers).
// X alone would take 67 us of the first (7.0 TB/s), X and the pivots in any order 77.
// A unit whose candidates are a quarter of all pairs and more is left alone, for screen_state to call dense: its rows share
// a direction (or a few columns), which the sketch cannot tell from being near.
// Two rows per lane group: the rows in flight on an XCD (256 workgroups of 8 at d = 4096) then stay about within one unit, whose
// pivots its L2 can hold; four rows spread over two units (STREAM, 28 x T=2048, d=4096: call 150 us against 143; 32 x T=8192:
// 632 against 619), one row starts more workgroups (145, 619).
// STREAM: see screen_streams.
template <typename In, int LPR, int UN, bool WHOLE, int PASSES, bool STREAM>
__global__ __launch_bounds__(256) void k_screen_exact(ScreenParams p, int row_blocks, int total) {
    __shared__ uint32_t s_pairs;
    const int per = (total + 7) >> 3;
    const int w = (int)(blockIdx.x & 7) * per + (int)(blockIdx.x >> 3);
    if (w >= total || (int)(blockIdx.x >> 3) >= per) return;
    const ScreenUnit U(p.T, p.nch, p.edge_cap);
    const int unit = w / row_blocks, rb = w - unit * row_blocks;
    int layer, group;
    char* base = screen_unit(p, U, unit, &layer, &group);
    const In* X = screen_x<In>(p, layer, group);
    const int32_t* piv = reinterpret_cast<const int32_t*>(base + U.o_piv);
    int32_t* size = reinterpret_cast<int32_t*>(base + U.o_size);
    float* rho = reinterpret_cast<float*>(base + U.o_rho);
    uint16_t* cl = reinterpret_cast<uint16_t*>(base + U.o_cl);
    const bool crowded = LPR == 64 && screen_crowded(p, base);
    if (threadIdx.x == 0) s_pairs = 0u;
    screen_barrier();
    const int li = threadIdx.x & (LPR - 1);
    const int t0 = rb * PASSES * (256 / LPR) + (int)threadIdx.x / LPR;
    // lane k of a group keeps what row k's sums are wanted for: they are looked at once, after the last row
    static_assert(PASSES <= LPR, "a lane per row");
    const int rows = 256 / LPR, mine = t0 + min(li, PASSES - 1) * rows, t_mine = min(mine, p.T - 1);
    const int q_mine = piv[t_mine];
    const float ss = rho[t_mine];
    int q[PASSES];
#pragma unroll
    for (int k = 0; k < PASSES; ++k) q[k] = PASSES == 1 ? q_mine : piv[min(t0 + k * rows, p.T - 1)];
    if (crowded) return;                                      // uniform
    const int qq = piv[q_mine];
    float xy = 0.f, xx = 0.f, yy = 0.f;
    uint32_t place = 0u, fl = 0u;
#pragma unroll
    for (int k = 0; k < PASSES; ++k) {
        // (a wave's row: scalars.  Shorter rows take the second product with themselves where they have no pivot, and not a branch.)
        const int t = LPR == 64 ? __builtin_amdgcn_readfirstlane(t0 + k * rows) : t0 + k * rows;
        const int s = LPR == 64 ? __builtin_amdgcn_readfirstlane(q[k]) : q[k];
        if (t < p.T) {
            const In *x = X + (size_t)t * (size_t)p.ld, *y = X + (size_t)s * (size_t)p.ld;
            float a, b, c;
            if (LPR < 64 || s != t) screen_products<In, LPR, STREAM, UN, WHOLE>(x, y, p.d, li, &a, &b, &c);
            else screen_products<In, LPR, STREAM, UN, WHOLE, false>(x, y, p.d, li, &a, &b, &c);
            if (li == k) { xy = a; xx = b; yy = c; }
        }
    }
    if (li < PASSES && mine < p.T) {
        const float r2 = xx > 0.f ? ss / xx : 1.f;            // (a zero row has no cosines: nothing to bound)
        rho[mine] = r2;
        if (p.inv_norm) p.inv_norm[mine] = xx > 0.f ? 1.0f / sqrtf(xx) : 0.f;
        fl |= r2 < p.f2 ? (uint32_t)SF_LOW : 0u;
        int c = mine;
        if (q_mine != mine && screen_cos(xy, xx, yy) >= p.cos_tight) {
            c = q_mine;
            if (qq != q_mine) fl |= SF_MESH;                  // the pivot may not be a member of its own cluster
            if (p.count_pairs) place = (uint32_t)atomicAdd(size + q_mine, 1) + 1u;   // pairs with the pivot and with earlier arrivals
        }
        cl[mine] = (uint16_t)c;
    }
    uint32_t* hdr = reinterpret_cast<uint32_t*>(base) + SU_PART + (blockIdx.x & 7) * 32;
    fl = (__ballot(fl & SF_LOW) != 0ull ? (uint32_t)SF_LOW : 0u) | (__ballot(fl & SF_MESH) != 0ull ? (uint32_t)SF_MESH : 0u);
    if (fl && (threadIdx.x & 63) == 0 && (__hip_atomic_load(hdr + SU_FLAGS, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & fl) != fl)
        atomicOr(hdr + SU_FLAGS, fl);
    if (!p.count_pairs) return;                               // uniform
    if (place) atomicAdd(&s_pairs, place);
    screen_barrier();
    if (threadIdx.x == 0 && s_pairs) atomicAdd(hdr + SU_PAIRS, s_pairs);
}

// Pairs inside the clusters of a unit, by 256 threads: how many tokens of its cluster came before, summed (in any order).
__device__ inline uint32_t screen_pairs_inside(const uint16_t* cl, int T) {
    extern __shared__ __align__(16) char lds[];               // [T] counts, two per word
    __shared__ uint32_t s_sum;
    uint32_t* count = reinterpret_cast<uint32_t*>(lds);
    const int tid = threadIdx.x;
    uint32_t sum = 0u;
    if (tid == 0) s_sum = 0u;
    for (int w = tid; w < (T + 1) / 2; w += 256) count[w] = 0u;
    __syncthreads();
    for (int t0 = tid; t0 < T; t0 += 256 * 8) {
        int c[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) c[u] = cl[min(t0 + 256 * u, T - 1)];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (t0 + 256 * u < T) sum += atomicAdd(&count[c[u] >> 1], 1u << (16 * (c[u] & 1))) >> (16 * (c[u] & 1)) & 0xFFFFu;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if ((tid & 63) == 0) atomicAdd(&s_sum, sum);
    __syncthreads();
    return s_sum;
}

// What a unit's counts say: every candidate is explained by a cluster (PLAIN); so many are not that the tiles behind are the better
// way (DENSE: p.open); or they are to be multiplied out (OPEN).
enum { UNIT_PLAIN, UNIT_OPEN, UNIT_DENSE };
__device__ inline int screen_state(const ScreenParams& p, const ScreenCounts& n) {
    return n.flags == 0u && n.cand == n.pairs ? UNIT_PLAIN : n.cand > n.pairs + p.open ? UNIT_DENSE : UNIT_OPEN;
}

// The candidates of an open unit that no cluster explains, by workgroup `slot` of `slots` (all threads; lanes: per product, a power of two; NB:
// blocks of 32 tokens at a time, 1 where a thread has 128 registers).  A round takes 128 x 128 tiles side by side, a power of two of them per
// workgroup and only as many as are needed for what is left: 256 threads of each find its pairs, all threads it has form the
// products (12 layers of T=512, d=768 in fp32, all tokens loose, with a workgroup per tile 88.7 -> 65.1 us and the walk).  Side by side they wait for
// each other, so a last round of few tiles, dealt to few workgroups four at a time, was as long as a whole one: 8 layers of T=2048, d=4096, all
// tokens loose 191 -> 184 us with a CU for every workgroup (one too many is a round more), 169 with sides by what is left; with 128 registers
// two workgroups of 512 threads share a CU: 28 layers of T=1000, d=2048 238 -> 218.  A tile's edges are counted in LDS and take
// their places in the unit's list with one atomic: one per edge, all to one address at 25 ns each, was most of this (T=2048, d=768 in
// fp32, clusters of five as wide as the threshold: 187 us).  Edges and counts go past the caches: the walk may be in the same launch.
struct RestTile {
    int n, edges, at, stop;
    uint32_t pair[SCREEN_TILE_PAIRS];
    uint2 edge[SCREEN_TILE_PAIRS];
    float rho[256];
    uint16_t cl[256];
};
template <int THREADS, int NB>
__device__ inline void screen_rest_tiles(const ScreenParams& p, const ScreenUnit& U, char* base, int layer, int group, bool low, int slot,
                                         int slots, int ntile, int lanes, bool f32, char* lds) {
    constexpr int SUB = THREADS / 256;
    RestTile* tiles = reinterpret_cast<RestTile*>(lds);
    uint32_t* hdr = reinterpret_cast<uint32_t*>(base);
    const float* rho = reinterpret_cast<const float*>(base + U.o_rho);
    const uint16_t* cl = reinterpret_cast<const uint16_t*>(base + U.o_cl);
    unsigned long long* edge = reinterpret_cast<unsigned long long*>(base + U.o_edge);
    for (int done = 0; done + slot < ntile;) {
        int side = 1;                                         // (uniform, the same in all of a unit's workgroups)
        while (side < SUB && side * slots < ntile - done) side *= 2;
        const int many = THREADS / side, sub = __builtin_amdgcn_readfirstlane((int)threadIdx.x / many), mine = (int)threadIdx.x & (many - 1);
        const int lane = mine & 63, l32 = lane & 31, half = lane >> 5, tile = done + sub * slots + slot;
        const bool exists = tile < ntile;                     // (uniform per tile; the barriers are everybody's)
        done += side * slots;
        RestTile& my = tiles[sub];
        int sb, tb;
        screen_blocks(min(tile, ntile - 1), &sb, &tb);
        __syncthreads();
        if (mine == 0) {
            my.n = my.edges = 0;
            if (sub == 0) tiles[0].stop = __hip_atomic_load(hdr + SU_DENSE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
        }
        if (mine < 256) {
            const int tok = min(mine < 128 ? sb * 128 + mine : tb * 128 + mine - 128, p.T - 1);
            my.rho[mine] = fminf(rho[tok], 1.f);
            my.cl[mine] = cl[tok];
        }
        __syncthreads();
        if (tiles[0].stop) break;                             // given up already (uniform)
        const ScreenTile me = screen_tile(p.T, sb, tb, __builtin_amdgcn_readfirstlane(mine >> 6));
        if (mine < 256 && me.any && exists) {
#pragma unroll 1
            for (int b0 = 0; b0 < 2; b0 += NB) {
                f32x16 acc[2][NB];
                screen_tile_products<NB>(base + U.o_z, p.T, p.nch, me, b0, acc);
#pragma unroll
                for (int bb = 0; bb < NB; ++bb) {
                    const int b = b0 + bb;
                    const int tl = me.t0 - tb * 128 + b * 32 + l32, t = tb * 128 + tl;
                    const int ct = my.cl[128 + tl];
                    auto row = [&](int i) { return me.s0 - sb * 128 + (i >> 4) * 32 + 4 * half + screen_row(i); };
                    uint64_t near = 0u;                           // bit 62 - 2 i: register i of the two blocks' 32
                    if (!low) {
                        near = (uint64_t)(screen_bits(acc[0][bb]) & SCREEN_BITS) << 32 | (screen_bits(acc[1][bb]) & SCREEN_BITS);
                    } else {                                      // some row holds little in its sketch: the pair's own bound
                        const float rt = my.rho[128 + tl];
#pragma unroll
                        for (int i = 0; i < 32; ++i) {
                            const float rs = my.rho[row(i)];
                            if (fabsf(acc[i >> 4][bb][i & 15]) >= 2.f ||
                                p.kap1 * sqrtf(rs * rt) + sqrtf((1.f - rs) * (1.f - rt)) + 1e-5f >= p.safe) near |= 1ull << (62 - 2 * i);
                        }
                    }
                    while (__builtin_amdgcn_ballot_w64(near != 0u) != 0ull)
                        if (near != 0u) {
                            const int i = __clzll((long long)near) >> 1, sl = row(i), s = sb * 128 + sl;
                            near &= ~(1ull << (62 - 2 * i));
                            if (s < t && t < p.T && my.cl[sl] != ct) {
                                const int n = atomicAdd(&my.n, 1);
                                if (n < SCREEN_TILE_PAIRS) my.pair[n] = (uint32_t)s << 16 | (uint32_t)t;
                            }
                        }
                }
            }
        }
        __syncthreads();
        int n = my.n;
        if (n > SCREEN_TILE_PAIRS) {                          // no saving in listing these
            if (mine == 0) __hip_atomic_store(hdr + SU_DENSE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            n = 0;
        }
        auto products = [&](auto lpr, auto in) {
            constexpr int LPR = decltype(lpr)::value;
            using In = decltype(in);
            const In* X = screen_x<In>(p, layer, group);
            const int li = mine & (LPR - 1);
            for (int k = mine / LPR; k < n; k += many / LPR) {
                const uint32_t e = my.pair[k];
                const int s = (int)(e >> 16), t = (int)(e & 0xFFFFu);
                float xy, xx, yy;
                screen_products<In, LPR>(X + (size_t)t * (size_t)p.ld, X + (size_t)s * (size_t)p.ld, p.d, li, &xy, &xx, &yy);
                const float c = screen_cos(xy, xx, yy);
                if (p.gamma && li == 0 && c > 0.f) atomicMax(reinterpret_cast<uint32_t*>(p.gamma) + t, __float_as_uint(c));
                if (li == 0 && c >= p.thr) my.edge[atomicAdd(&my.edges, 1)] = uint2{e, __float_as_uint(c)};
            }
        };
        auto pick = [&](auto in) {
            if (lanes == 64) products(std::integral_constant<int, 64>{}, in);
            else if (lanes == 32) products(std::integral_constant<int, 32>{}, in);
            else if (lanes == 16) products(std::integral_constant<int, 16>{}, in);
            else products(std::integral_constant<int, 8>{}, in);
        };
        if (f32) pick(float{});
        else pick(uint16_t{});
        __syncthreads();
        const int ne = my.edges;
        if (mine == 0 && ne > 0) my.at = (int)atomicAdd(hdr + SU_EDGES, (uint32_t)ne);
        __syncthreads();
        const int at = my.at;
        for (int k = mine; k < ne; k += many)
            if (at + k < U.edge_cap)
                __hip_atomic_store(edge + at + k, (unsigned long long)my.edge[k].y << 32 | my.edge[k].x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (mine == 0 && ne > 0 && at + ne > U.edge_cap) __hip_atomic_store(hdr + SU_DENSE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Groups that the sign-offs of a unit's workgroups come in: a word takes one every 25 ns, and most arrive together.  With one word for all
// workgroups of a sequence the walk started up to 12 us late: 28 layers of T=1000, d=2048 (505 workgroups), one token in fifty loose 128.8 -> 121.5 us.
constexpr int SIGN_OFFS = 32;
__device__ inline int screen_groups(int rest) { return min((rest + SIGN_OFFS - 1) / SIGN_OFFS, 8); }   // (a line of the header each)

// Whether this workgroup is the last one of a sequence (all threads): what the others stored is seen from here on.  A unit's workgroup `slot` of
// `rest` signs off in its group's word of the unit's header (zero since the sketches), the last one of a group adds one to `counter`, and
// the workgroup that knows how many groups there are (hdr: NULL) takes their number off: whoever leaves zero is the last, and zero is what the next call needs.
__device__ inline bool screen_last(int32_t* counter, uint32_t* hdr, int slot, int rest, int n_groups) {
    __shared__ int s_last;
    drain_stores();
    __syncthreads();
    if (threadIdx.x == 0) {
        if (hdr) {
            const int groups = screen_groups(rest), k = slot % groups, members = (rest - k + groups - 1) / groups;
            s_last = (int)atomicAdd(hdr + SU_PART + k * 32 + SU_DONE, 1u) == members - 1 && atomicAdd(counter, 1) == -1;
        } else s_last = atomicAdd(counter, -n_groups) == n_groups;
        if (s_last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    return s_last;
}

// k_screen_rest: the unexplained candidates of all units as a launch of its own, where the pairs inside clusters are counted
// here (rows of fewer than 128 pieces: LPR is 8 or 16).  Units without any are left at once.  (LPR and In as arguments, which costs
// registers: 144 units of T=701, d=64, one token in fifty loose 75.5 -> 84.4 us.)
template <typename In, int LPR>
__global__ __launch_bounds__(256) void k_screen_rest(ScreenParams p, int ntile) {
    __shared__ RestTile tile;
    const ScreenUnit U(p.T, p.nch, p.edge_cap);
    const int units = p.G * p.L, unit = (int)blockIdx.x % units;
    int layer, group;
    char* base = screen_unit(p, U, unit, &layer, &group);
    uint32_t* hdr = reinterpret_cast<uint32_t*>(base);
    ScreenCounts n_unit = screen_counts(hdr);
    n_unit.pairs = screen_pairs_inside(reinterpret_cast<const uint16_t*>(base + U.o_cl), p.T);
    if ((int)blockIdx.x < units && threadIdx.x == 0) hdr[SU_PART + SU_PAIRS] = n_unit.pairs;   // (where the exact pass leaves its counts)
    const int state = screen_state(p, n_unit);
    if (state == UNIT_DENSE && (int)blockIdx.x < units && threadIdx.x == 0)
        __hip_atomic_store(hdr + SU_DENSE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (state == UNIT_OPEN)
        screen_rest_tiles<256, 2>(p, U, base, layer, group, (n_unit.flags & SF_LOW) != 0u, (int)blockIdx.x / units, (int)gridDim.x / units, ntile, LPR,
                                  sizeof(In) == 4, reinterpret_cast<char*>(&tile));
}

// ------------------------------------------------------------------------------------------------
// k_screen_chain: the layers, one after the other, on clusters and edges.  One workgroup per sequence; a wave owns U words of
// the set, 64 tokens each, and their membership stays in registers from layer to layer.  Without edges a layer is: every
// inherited token puts its id under an integer minimum of its cluster (the earliest inherited member is the only valid one),
// one barrier, every token looks its cluster up, and the new set leaves as ballots (one bit per token).  Cluster slots carry a
// layer stamp that falls from layer to layer, so they need no clearing, and there are two sets of them in turns, so that one
// barrier per layer is enough.  Index lists, counts and Gram operations follow from the bits of a layer and the one before: the
// launch behind writes them, for all layers at once.
// Bound by the instructions of a wave (about 45 and 22 per token of a lane) and two trips to LDS per layer: nothing else is
// in the loop.  The clusters come from memory D layers ahead, straight into registers, as buffer loads (a lane address and a
// scalar one, past the last token zero); tokens outside the set put their id in a place of their own, which takes less than a
// branch around the minimum; a lane stores a word.  Clusters by way of LDS, all of them there before the first layer, and
// predicated minima took, us: 12 x T=512 7.7 (now 4.7), 28 x T=2048 24.6 (12.4), 8 x T=8192 24.2 (12.7), 16 x T=12000 77.9 (42.7).
struct ChainParams {
    ScreenParams s;
    int earlier_only;
    int32_t* idx;              // row 0 of the call's outputs (sequence 0); rows T apart
    int32_t* counts;
    unsigned long long* ops;
    int32_t* adds;             // may be NULL
    int32_t* removes;          // may be NULL
    long long list_gs, counts_gs, ops_gs;   // elements between sequences
    // nearest representative of every token (Section 2.3), if wanted (one sequence): row 0 of the call's outputs, rows T and
    // 8 apart; pos: the representative's position in its set
    int32_t* assign;
    int32_t* pos;
    int32_t* info;
    int f32;                   // rows are fp32 (else bf16)
    int rest, ntile, lanes;    // workgroups per unit for the unexplained candidates (0: a launch of their own was), see screen_rest_tiles
};

constexpr int LIST_WORDS = FUSED_MAX_T / 64;
constexpr int LIST_SCRATCH = LIST_WORDS * (3 * 4 + 2 * 8);    // LDS that writing a layer's lists takes: places per word, the set's words and the ones before
// ... and its assignment (screen_assign): two words per token besides
constexpr int assign_lds(int T) { return LIST_SCRATCH + (T + 63) / 64 * 64 * 8; }
static_assert(assign_lds(FUSED_MAX_T) <= CHAIN_LDS, "LDS of a layer's lists and assignment");

// LDS of the walk: two sets of cluster slots, marks (edges only).
template <int THREADS, int U>
__host__ __device__ constexpr int chain_lds(int T) {
    constexpr int tokens = THREADS * U, walk = (tokens + 64) * 8 + tokens, rest = THREADS / 256 * (int)sizeof(RestTile), most = walk > rest ? walk : rest;
    return most > assign_lds(T) ? most : assign_lds(T);
}
static_assert(chain_lds<1024, 16>(FUSED_MAX_T) <= CHAIN_LDS, "LDS of the walk");

constexpr int CHAIN_BUFFER = 0x00020000;                      // a buffer of plain bytes: loads past its end give zero, stores are dropped
typedef int i32x2 __attribute__((ext_vector_type(2)));
__device__ int chain_writelane(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");   // (has no builtin)

// Token u of a lane: a wave owns U words of a layer's set, side by side.
template <int U> __device__ inline int chain_token(int u) {
    int t = ((int)threadIdx.x >> 6) * (U * 64) + ((int)threadIdx.x & 63);
    if constexpr (U > 8) asm volatile("" : "+v"(t));          // (what is formed from all of a lane's tokens in advance is more than there are registers)
    return t + 64 * u;
}

// One layer's lists, counts and Gram operations from the bits of its set and of the one before (any workgroup size up to
// 1024; scratch: LIST_SCRATCH bytes of LDS); part of parts: its share of the tokens.  One wave reads the bits and sums over
// the words before; they stay in LDS for the others.  (Read from memory by each of them again, behind the stores of the tokens
// before, and a layer by one workgroup: 28 layers of T=2048 7.0 us, now 5.5, 8 layers of four sequences of T=8192 11.4, now 7.1.)
struct ListScratch {
    unsigned long long *now, *was;                            // [words] the set, and the one inherited
    int* start;                                               // [3][LIST_WORDS] members in the words before: the set, added, removed
    __device__ explicit ListScratch(int* scratch) {
        now = reinterpret_cast<unsigned long long*>(scratch);
        was = now + LIST_WORDS;
        start = reinterpret_cast<int*>(was + LIST_WORDS);
    }
};
__device__ inline int list_rank(unsigned long long m) {       // members before this lane
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}
__device__ inline void screen_lists(const ChainParams& c, const ScreenUnit& SU, int l, int g, int* scratch, int part = 0, int parts = 1) {
    const ScreenParams& p = c.s;
    const int T = p.T, words = (T + 63) >> 6, tid = threadIdx.x, lane = tid & 63;
    const ListScratch s(scratch);
    const bool full = p.first + l == 0;
    const size_t row = (size_t)(p.first + l);
    if (tid < 64) {                                           // one wave: prefix sums over the words
        const char* unit = p.area + (long long)g * p.area_gs + (long long)l * SU.bytes;
        const unsigned long long* now = reinterpret_cast<const unsigned long long*>(unit + SU.o_mask);
        const unsigned long long* was = l > 0 ? reinterpret_cast<const unsigned long long*>(unit - SU.bytes + SU.o_mask) : now + words;
        int tot[3] = {0, 0, 0};
        for (int w0 = 0; w0 < words; w0 += 64) {
            const int w = w0 + lane;
            const unsigned long long a = w < words ? now[w] : 0ull, b = w < words && !full ? was[w] : 0ull;
            const unsigned long long m[3] = {a, a & ~b, b & ~a};
            if (w < words) { s.now[w] = a; s.was[w] = b; }
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const int pc = __popcll(m[k]);
                int inc = pc;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int x = __shfl_up(inc, o, 64);
                    if (lane >= o) inc += x;
                }
                if (w < words) s.start[k * LIST_WORDS + w] = tot[k] + inc - pc;
                tot[k] += __builtin_amdgcn_readlane(inc, 63);
            }
        }
        if (lane == 0 && part == 0) {
            const unsigned long long TT = (unsigned long long)T, rr = (unsigned long long)(tot[0] - tot[1] + tot[2]);   // (kept ones and the removed)
            *reinterpret_cast<int4*>(c.counts + (long long)g * c.counts_gs + row * 4) =
                full ? int4{tot[0], tot[0], 0, ADA_OK} : int4{tot[0], tot[1], tot[2], ADA_OK};
            c.ops[(long long)g * c.ops_gs + row] = full ? TT * TT : rr * rr + (TT - rr) * (rr - (unsigned long long)tot[2]);   // Table 6 / eq. (6)
        }
    }
    screen_barrier();
    int32_t* idx = c.idx + (long long)g * c.list_gs + row * T;
    int32_t* adds = c.adds && !full ? c.adds + (long long)g * c.list_gs + row * T : nullptr;
    int32_t* removes = c.removes && !full ? c.removes + (long long)g * c.list_gs + row * T : nullptr;
    for (int t = part * (int)blockDim.x + tid; t < words * 64; t += parts * (int)blockDim.x) {
        const int w = __builtin_amdgcn_readfirstlane(t >> 6);
        const unsigned long long a = s.now[w], b = s.was[w];
        auto put = [&](int32_t* dst, int k, unsigned long long m) {
            if (dst && ((m >> lane) & 1ull)) dst[s.start[k * LIST_WORDS + w] + list_rank(m)] = t;
        };
        put(idx, 0, a);
        put(adds, 1, a & ~b);
        put(removes, 2, b & ~a);
    }
    screen_barrier();
}

// f(both ends) for every edge.
template <int THREADS, typename F>
__device__ inline void chain_each(uint32_t n_edge, const uint2* edge, F f) {
    for (uint32_t e = threadIdx.x; e < n_edge; e += THREADS) {
        const uint32_t v = edge[e].x;
        f((int)(v >> 16), (int)(v & 0xFFFFu));
    }
}

// Whether a layer with edges has a token outside the set that no representative is within the threshold of: neither its
// cluster nor an edge leads to a member of the set.  (Definition 2.2 compares with all earlier tokens, and step 5 drops an
// inherited token that any earlier inherited one hits, so on a chain a ~ b ~ c with a not ~ c both b and c leave the set,
// and so do the members of b's or c's cluster.)  All threads, after the set is known; leaves marks, and slots of this layer
// that say nothing about it any more.
template <int THREADS, int U>
__device__ inline bool chain_alone(uint32_t n_edge, const uint2* edge, uint32_t stamp, uint32_t* slot, uint8_t* mark,
                                   const int (&cid)[U], const unsigned long long (&in)[U], int T) {
    const int lane = (int)threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int t = chain_token<U>(u);
        slot[cid[u]] = 0xFFFFFFFFu;
        if (t < T) mark[t] = (in[u] >> lane) & 1ull ? 1 : 0;
    }
    screen_barrier();
#pragma unroll
    for (int u = 0; u < U; ++u)
        if ((in[u] >> lane) & 1ull) slot[cid[u]] = stamp;
    chain_each<THREADS>(n_edge, edge, [&](int s, int t) {     // (a member's mark is read, only the others' are written)
        if ((mark[s] & 1) && !(mark[t] & 1)) mark[t] = 2;
        if ((mark[t] & 1) && !(mark[s] & 1)) mark[s] = 2;
    });
    screen_barrier();
    int alone = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int t = chain_token<U>(u);
        alone |= t < T && slot[cid[u]] != stamp && mark[min(t, T - 1)] == 0;
    }
    return __syncthreads_or(alone) != 0;
}

// A layer that has edges (all threads; the marks are zero on entry, barriers inside; on return some marks are set).  The barriers are for
// LDS alone, so that the next layer's clusters come in behind this one's edges: each layer with edges asked for its own and, behind
// them, for those of the D layers after it, and waited for both: 28 layers of T=300, d=768 78.9 -> 73.9 us, of T=2048, d=4096 239 -> 229 (one
// token in fifty loose).
template <int THREADS, int U>
__device__ inline void chain_edges(bool full, int earlier_only, uint32_t n_edge, const uint2* edge, uint32_t stamp,
                                   uint32_t* slot, uint8_t* mark, const int (&cid)[U], unsigned long long (&in)[U], int T) {
    const int lane = (int)threadIdx.x & 63;
    if (full) {                                               // Definition 2.2: no earlier token within the threshold
        chain_each<THREADS>(n_edge, edge, [&](int, int t) { mark[t] = 2; });
        screen_barrier();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = chain_token<U>(u);
            in[u] = __ballot(t < T && cid[u] == t && !(mark[min(t, T - 1)] & 2));
        }
        screen_barrier();
        return;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int t = chain_token<U>(u);
        const bool inh = (in[u] >> lane) & 1ull;
        if (inh) atomicMin(&slot[cid[u]], stamp | (uint32_t)t);
        if (t < T) mark[t] = inh ? 1 : 0;
    }
    screen_barrier();
    // step 5 along edges: an earlier inherited token hits a later one (only bit 1 is read, only bit 2 set here)
    chain_each<THREADS>(n_edge, edge, [&](int s, int t) { if ((mark[s] & 1) && (mark[t] & 1)) mark[t] = 3; });
    screen_barrier();
    uint32_t low[U];                                          // earliest inherited member of the token's cluster (or none)
    unsigned long long keep[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int t = chain_token<U>(u);
        const uint32_t v = slot[cid[u]];
        low[u] = (v & 0xFFFFC000u) == stamp ? v & 0x3FFFu : 0xFFFFFFFFu;
        keep[u] = __ballot(((in[u] >> lane) & 1ull) && low[u] == (uint32_t)t && mark[min(t, T - 1)] != 3);
    }
    screen_barrier();
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (chain_token<U>(u) < T) mark[chain_token<U>(u)] = (keep[u] >> lane) & 1ull ? 4 : 0;
    screen_barrier();
#pragma unroll
    for (int u = 0; u < U; ++u)                               // the cluster's earliest inherited member covers only if valid
        if (low[u] != 0xFFFFFFFFu && mark[low[u]] != 4) low[u] = 0xFFFFFFFFu;
    screen_barrier();
    chain_each<THREADS>(n_edge, edge, [&](int s, int t) {     // steps 7-8 along edges (valid tokens keep their mark)
        if (mark[s] & 4) { if (!(mark[t] & 4)) mark[t] = 8; }
        if ((mark[t] & 4) && !earlier_only) { if (!(mark[s] & 4)) mark[s] = 8; }
    });
    screen_barrier();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int t = chain_token<U>(u);
        const bool covered = (low[u] != 0xFFFFFFFFu && !(earlier_only && low[u] > (uint32_t)t)) || mark[min(t, T - 1)] == 8;
        in[u] = keep[u] | (__ballot(t < T && !covered) & ~in[u]);        // steps 9 and 10
    }
    screen_barrier();
}

// The nearest representative of every token of a layer: all representatives within the threshold of a token are members
// of its cluster or joined to it by an edge, so if there is one the largest |cos| is among these; usually there is just one
// and nothing has to be multiplied.  Layers with a token that has none (chain_alone; only layers with edges can) do not come
// here: their assignment takes the products with the whole set, on the tiles of k_cascade_rest.  (any workgroup size up to
// 1024; scratch: assign_lds(T) bytes of LDS)
__device__ inline void screen_assign(const ChainParams& c, const ScreenUnit& SU, int l, int g, int* scratch, int part = 0, int parts = 1) {
    const ScreenParams& p = c.s;
    const int T = p.T, words = (T + 63) >> 6, tid = threadIdx.x, nthr = blockDim.x, lane = tid & 63;
    char* unit = p.area + (long long)g * p.area_gs + (long long)l * SU.bytes;
    const unsigned long long* now = reinterpret_cast<const unsigned long long*>(unit + SU.o_mask);
    const uint16_t* cl = reinterpret_cast<const uint16_t*>(unit + SU.o_cl);
    const uint2* edge = reinterpret_cast<const uint2*>(unit + SU.o_edge);
    const int n_edge = (int)reinterpret_cast<const uint32_t*>(unit)[SU_EDGES];
    if (n_edge > 0 && part > 0) return;                       // (uniform; with edges one workgroup sees to all tokens)
    const size_t row = (size_t)(p.first + l);
    int32_t* assign = c.assign + row * T;
    int32_t* pos = c.pos + row * T;
    const ListScratch ls(scratch);                            // (start: representatives in the words before)
    uint32_t* member = reinterpret_cast<uint32_t*>(scratch) + LIST_SCRATCH / 4;    // [64 words] earliest representative of a cluster
    uint32_t* n_member = member + words * 64;                 // [64 words] how many it has
    for (int t = tid; t < words * 64; t += nthr) { member[t] = 0xFFFFFFFFu; n_member[t] = 0u; }
    if (tid < 64) {
        int tot = 0;
        for (int w0 = 0; w0 < words; w0 += 64) {
            const unsigned long long a = w0 + lane < words ? now[w0 + lane] : 0ull;
            const int pc = __popcll(a);
            int inc = pc;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int x = __shfl_up(inc, o, 64);
                if (lane >= o) inc += x;
            }
            if (w0 + lane < words) { ls.now[w0 + lane] = a; ls.start[w0 + lane] = tot + inc - pc; }
            tot += __builtin_amdgcn_readlane(inc, 63);
        }
        if (lane == 0 && part == 0) *reinterpret_cast<int4*>(c.info + row * 8) = int4{T - tot, 0, 0, ADA_OK};
    }
    __syncthreads();
    auto is_in = [&](int t) { return (ls.now[t >> 6] >> (t & 63)) & 1ull; };
    auto put = [&](int t, int a) {
        assign[t] = a;
        pos[t] = ls.start[a >> 6] + __popcll(ls.now[a >> 6] & ((1ull << (a & 63)) - 1ull));
    };
    for (int t = tid; t < T; t += nthr)
        if (is_in(t)) {
            atomicMin(&member[cl[t]], (uint32_t)t);
            if (n_edge) atomicAdd(&n_member[cl[t]], 1u);
        }
    __syncthreads();
    if (n_edge == 0) {
        for (int t0 = part * 4 * nthr + tid; t0 < T; t0 += parts * 4 * nthr) {   // (a load behind a store waits for it)
            int ct[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) ct[u] = cl[min(t0 + u * nthr, T - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int t = t0 + u * nthr;
                if (t < T) put(t, is_in(t) ? t : (int)min(member[ct[u]], (uint32_t)(T - 1)));
            }
        }
        __syncthreads();
        return;
    }
    // With edges: the usual packed key per token, (bits of |cos|) << 32 | INT_MAX - id, in the unit's memory for sizes and rho
    unsigned long long* key = reinterpret_cast<unsigned long long*>(unit + SU.o_size);
    for (int t = tid; t < T; t += nthr) __hip_atomic_store(key + t, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    for (int e = tid; e < n_edge; e += nthr) {
        const uint2 v = edge[e];
        const int s = (int)(v.x >> 16), t = (int)(v.x & 0xFFFFu);
        const unsigned long long hi = (unsigned long long)v.y << 32;
        if (is_in(s) && !is_in(t)) atomicMax(key + t, hi | (uint32_t)(INT_MAX - s));
        if (is_in(t) && !is_in(s)) atomicMax(key + s, hi | (uint32_t)(INT_MAX - t));
    }
    drain_stores();
    __syncthreads();
    // tokens that an edge or several members of their cluster compete for: the members' products, one wave per token
    for (int w = tid >> 6; w < words; w += nthr >> 6) {
        const int tt = w * 64 + lane;
        const bool mine = tt < T && !is_in(min(tt, T - 1));
        const uint32_t nm = tt < T ? n_member[cl[tt]] : 0u;
        const unsigned long long k = mine ? __hip_atomic_load(key + tt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
        if (tt < T && !mine) put(tt, tt);
        if (mine && nm == 0u && k != 0ull) put(tt, INT_MAX - (int)(uint32_t)k);
        if (mine && nm == 1u && k == 0ull) put(tt, (int)member[cl[tt]]);
        unsigned long long open = __ballot(mine && nm > 0u && (nm > 1u || k != 0ull));
        while (open) {
            const int j = __builtin_amdgcn_readfirstlane(__ffsll((long long)open) - 1), t = w * 64 + j;
            open &= open - 1ull;
            unsigned long long best = ((unsigned long long)(uint32_t)__shfl((int)(k >> 32), j, 64) << 32) | (uint32_t)__shfl((int)(uint32_t)k, j, 64);
            const int ct = cl[t];
            for (int v = 0; v < words; ++v) {
                const int s = v * 64 + lane;
                unsigned long long m = __ballot(s < T && is_in(min(s, T - 1)) && cl[min(s, T - 1)] == ct);
                for (; m; m &= m - 1ull) {
                    const int q = v * 64 + __ffsll((long long)m) - 1;
                    float xy, xx, yy;
                    if (c.f32) {
                        const float* X = screen_x<float>(p, l, g);
                        screen_products<float, 64>(X + (size_t)t * (size_t)p.ld, X + (size_t)q * (size_t)p.ld, p.d, lane, &xy, &xx, &yy);
                    } else {
                        const uint16_t* X = screen_x<uint16_t>(p, l, g);
                        screen_products<uint16_t, 64>(X + (size_t)t * (size_t)p.ld, X + (size_t)q * (size_t)p.ld, p.d, lane, &xy, &xx, &yy);
                    }
                    const unsigned long long cand = ((unsigned long long)__float_as_uint(screen_cos(xy, xx, yy)) << 32) | (uint32_t)(INT_MAX - q);
                    best = cand > best ? cand : best;
                }
            }
            if (lane == 0) put(t, INT_MAX - (int)(uint32_t)best);
        }
    }
    __syncthreads();
}

__device__ inline unsigned long long uniform64(unsigned long long v) {
    return (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32 | (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
}

// Workgroups of the walk's launch that a CU holds at once: registers.  (Up to 512 tokens a unit's tiles have a workgroup each, on CUs of
// their own, and the registers are worth more.)
template <int THREADS, int U> constexpr int chain_places() { return THREADS == 512 && U > 1 ? 2 : 1; }
template <int THREADS, int U, int D>
__global__ __launch_bounds__(THREADS, (THREADS / 256 * chain_places<THREADS, U>())) void k_screen_chain(ChainParams c) {
    extern __shared__ __align__(16) char lds[];
    static_assert(SCREEN_MAX_LAYERS == 64, "a lane per layer");
    constexpr int TOKENS = THREADS * U, SET = TOKENS + 64;
    unsigned long long alone = 0ull;                          // layers whose assignment is left to the tiles (uniform)
    const ScreenParams& p = c.s;
    const ScreenUnit SU(p.T, p.nch, p.edge_cap);
    const int tid = threadIdx.x, T = p.T, lane = tid & 63, words = (T + 63) >> 6;
    int g = blockIdx.x;
    const bool walker = g < p.G;
    // Workgroups from G on see to the unexplained candidates of a unit each.  Where there are any, the last one of a sequence to be done
    // walks (its walker counts as one of them): nobody waits for anybody.  (As a launch of its own in front of the walk they took 2.4 to
    // 4.8 us, and 3 us of the host, to find nothing: calls of 12 x T=512, d=768 in fp32 28.8 -> 25.6 us, 12 x T=2048, d=768 39.9 -> 37.6, 28 x
    // T=2048, d=4096 128.4 -> 126.7.  With one token in ten loose, and all of them, a launch of their own with the walk of that time -> now: 16 x T=300, d=256
    // 51.4 -> 52.6 and 66.5 -> 64.8, 12 x T=512 60.3 -> 55.5 and 105.5 -> 83.5, 12 x T=1000 60.6 -> 60.8 and 87.6 -> 85.9, 12 x T=2048, d=768 96.4 -> 83.3
    // and 148 -> 117, 28 x T=2048, d=4096 285 -> 260 and 665 -> 543, 4 x T=8192, d=512 220 -> 152 and 240 -> 191.)
    if (!walker) {
        const int units = p.G * p.L, b = g - p.G;
        int layer;
        char* base = screen_unit(p, SU, b % units, &layer, &g);
        __shared__ int s_unit;
        if (tid < 64) {
            const ScreenCounts n = screen_counts(reinterpret_cast<const uint32_t*>(base));
            s_unit = screen_state(p, n) | ((n.flags & SF_LOW) ? 16 : 0);
        }
        screen_barrier();
        const int state = __builtin_amdgcn_readfirstlane(s_unit);
        if ((state & 15) != UNIT_OPEN) return;
        screen_rest_tiles<THREADS, THREADS / 256 * chain_places<THREADS, U>() < 4 ? 2 : 1>(p, SU, base, layer, g, (state & 16) != 0, b / units, c.rest, c.ntile, c.lanes, c.f32 != 0, lds);
        if (!screen_last(reinterpret_cast<int32_t*>(reinterpret_cast<char*>(p.meta) + (long long)g * p.area_gs) + META_WALK, reinterpret_cast<uint32_t*>(base), b / units, c.rest, 0)) return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    uint32_t* slots = reinterpret_cast<uint32_t*>(lds);       // [2][SET] stamp << 14 | earliest inherited member; the last 64 take what is none
    uint8_t* mark = reinterpret_cast<uint8_t*>(lds + SET * 8);    // bits: 1 inherited, 2 hit by an earlier inherited token, 4 valid, 8 covered
    int32_t* meta = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(p.meta) + (long long)g * p.area_gs);
    char* area = p.area + (long long)g * p.area_gs;
    auto unit_of = [&](int l) { return area + (uint32_t)l * (uint32_t)SU.bytes; };   // (a sequence's area is 34 MB at most)
    auto mask_of = [&](int l) { return reinterpret_cast<unsigned long long*>(unit_of(l) + SU.o_mask); };
    auto tok = [](int u) { return chain_token<U>(u); };
    auto clusters = [&](int l, int (&cid)[U]) {               // (past the last token: zero, a slot like any other)
        const auto row = __builtin_amdgcn_make_buffer_rsrc(unit_of(l) + SU.o_cl, 0, 2 * T, CHAIN_BUFFER);
#pragma unroll
        for (int u = 0; u < U; ++u) cid[u] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(row, 2 * tok(u), 0, 0);
    };
    int ahead[D][U], cid[U];
    const int skip = p.first == 0 ? 1 : 0;
    clusters(0, cid);
#pragma unroll
    for (int k = 0; k < D; ++k) clusters(min(skip + k, p.L - 1), ahead[k]);
    int loaded = skip;                                        // the layer that ahead[0] belongs to

    const int progress = meta[META_PROGRESS];
    const uint32_t* hdr = reinterpret_cast<const uint32_t*>(area + (long long)min(lane, p.L - 1) * SU.bytes);   // of the layer with this lane's number
    uint32_t edges_of = 0u;
    bool is_dense = false;
    auto look = [&] {
        edges_of = __hip_atomic_load(hdr + SU_EDGES, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        is_dense = __hip_atomic_load(hdr + SU_DENSE, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
    };
    if (!walker) look();                                      // (in flight beside the counts)
    unsigned long long open = 0ull, closed = 0ull;            // layers with unexplained candidates; with too many of them
    if (c.rest) {                                             // (one wave looks: sixteen took 3 us longer over 28 layers' lines)
        __shared__ unsigned long long s_state[2];
        if (wave == 0) {
            const int state = screen_state(p, screen_counts(hdr));
            open = __ballot(lane < p.L && state == UNIT_OPEN);
            closed = __ballot(lane < p.L && state == UNIT_DENSE);
            if (lane == 0) { s_state[0] = open; s_state[1] = closed; }
        }
        screen_barrier();
        open = uniform64(s_state[0]);
        closed = uniform64(s_state[1]);
    }
    if (walker && open && !screen_last(meta + META_WALK, nullptr, 0, 0, __popcll(open) * screen_groups(c.rest))) return;   // uniform
    if (walker && (open || !c.rest)) look();                  // (plain units have neither)
    const unsigned long long dense = __ballot(lane < p.L && (is_dense || ((closed >> lane) & 1ull)));
    const unsigned long long edged = __ballot(lane < p.L && edges_of != 0u);
    for (int t = tid; t < 2 * SET; t += THREADS) slots[t] = 0xFFFFFFFFu;
    for (int t = tid; t < TOKENS; t += THREADS) mark[t] = 0;
    // membership, one bit per lane and u; a lane whose token does not exist is a member of nothing
    unsigned long long in[U];
#pragma unroll
    for (int u = 0; u < U; ++u) in[u] = 0ull;
    auto exists = [&](int u) {                                // (uniform: bits of word u's tokens)
        const int n = T - (wave * U + u) * 64;
        return n >= 64 ? ~0ull : n > 0 ? (1ull << n) - 1ull : 0ull;
    };
    const int word_at = lane < U ? (wave * U + lane) * 8 : INT_MAX;   // lane u stores word u of its wave
    auto put = [&](unsigned long long* mask) {
        i32x2 v = {0, 0};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            v[0] = chain_writelane((int)(uint32_t)in[u], u, v[0]);
            v[1] = chain_writelane((int)(uint32_t)(in[u] >> 32), u, v[1]);
        }
        __builtin_amdgcn_raw_buffer_store_b64(v, __builtin_amdgcn_make_buffer_rsrc(mask, 0, 8 * words, CHAIN_BUFFER), word_at, 0, 0);
    };
    if (p.first > 0) {                                        // go on from the set an earlier launch left
        if (progress != p.first) {
            if (tid == 0) *reinterpret_cast<unsigned long long*>(meta + META_ALONE) = 0ull;
            return;
        }
        __syncthreads();
        const int32_t* idx = c.idx + (long long)g * c.list_gs + (size_t)(p.first - 1) * T;
        const int r = c.counts[(long long)g * c.counts_gs + (size_t)(p.first - 1) * 4];
        for (int j = tid; j < r; j += THREADS) mark[idx[j]] = 1;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; ++u) in[u] = __ballot(tok(u) < T && mark[tok(u)] != 0);
        put(mask_of(0) + words);
    }
    __syncthreads();
    int i = 0;
    bool stop = false;
    while (i < p.L) {
        if ((dense >> i) & 1ull) { stop = true; break; }      // uniform
        const bool has_edges = (edged >> i) & 1ull;
        if (has_edges || p.first + i == 0) {
            if (loaded == i) {
#pragma unroll
                for (int u = 0; u < U; ++u) cid[u] = ahead[0][u];
            } else if (i > 0 || p.first > 0) clusters(i, cid);
            if (has_edges) {
                if (loaded != i + 1) {
                    loaded = -1;
                    if ((edged >> i) & 2ull) { clusters(i + 1, ahead[0]); loaded = i + 1; }   // (in flight behind the edges)
                }
                const uint32_t n_edge = (uint32_t)__builtin_amdgcn_readlane((int)edges_of, i);
                const uint32_t stamp = (uint32_t)(0x3FFFE - i) << 14;
                uint32_t* slot = slots + (i & 1 ? SET : 0);
                const uint2* edge = reinterpret_cast<const uint2*>(area + (long long)i * SU.bytes + SU.o_edge);
                screen_barrier();
                chain_edges<THREADS, U>(p.first + i == 0, c.earlier_only, n_edge, edge, stamp, slot, mark, cid, in, T);
                if (c.assign && chain_alone<THREADS, U>(n_edge, edge, stamp, slot, mark, cid, in, T)) alone |= 1ull << i;
                for (int t = tid; t < TOKENS; t += THREADS) mark[t] = 0;
                screen_barrier();
            } else {                                          // Definition 2.2: a cluster's pivot is earlier than its other members
#pragma unroll
                for (int u = 0; u < U; ++u) in[u] = __ballot(cid[u] == tok(u)) & exists(u);
            }
            put(mask_of(i));
            ++i;
            continue;
        }
        const unsigned long long other = (dense | edged) >> i;
        const int end = other ? min(p.L, i + __builtin_ctzll(other)) : p.L;
        if (loaded != i) {
#pragma unroll
            for (int k = 0; k < D; ++k) clusters(min(i + k, p.L - 1), ahead[k]);
        }
        const int first_set = i & 1;
        while (i < end) {
#pragma unroll
            for (int k = 0; k < D; ++k) {
                if (i >= end) break;
                uint32_t* slot = slots + ((D % 2 ? i & 1 : (first_set + k) & 1) ? SET : 0);   // (D even: always the same for ahead[k])
                const uint32_t stamp = (uint32_t)(0x3FFFE - i) << 14;   // (the empty slot's own stamp is 0x3FFFF)
                uint32_t v[U];
#pragma unroll
                for (int u = 0; u < U; ++u)
                    atomicMin(&slot[__builtin_amdgcn_inverse_ballot_w64(in[u]) ? ahead[k][u] : TOKENS + lane], stamp | (uint32_t)tok(u));
                screen_barrier();
#pragma unroll
                for (int u = 0; u < U; ++u) v[u] = slot[ahead[k][u]] - stamp;   // this layer's stamp is the smallest so far
                clusters(min(i + D, p.L - 1), ahead[k]);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const unsigned long long valid = __ballot(v[u] == (uint32_t)tok(u));   // step 5 (only inherited tokens were there)
                    const unsigned long long covered = __ballot(v[u] < (c.earlier_only ? (uint32_t)tok(u) : 0x4000u));   // steps 7-8
                    in[u] = valid | (exists(u) & ~covered);   // steps 9 and 10
                }
                put(mask_of(i));
                ++i;
            }
        }
        loaded = -1;
    }
    // lists that the launch behind reads; all of them if it needs the units' memory for its hit table
    if (stop || alone != 0ull) {
        __syncthreads();
        for (int l = 0; l < i; ++l) {
            const bool tiles = (alone >> l) & 1ull;
            if (stop || tiles) screen_lists(c, SU, l, g, reinterpret_cast<int*>(lds));
            if (stop && c.assign && !tiles) screen_assign(c, SU, l, g, reinterpret_cast<int*>(lds));
        }
    }
    if (tid == 0) {
        meta[META_PROGRESS] = p.first + i;
        *reinterpret_cast<unsigned long long*>(meta + META_ALONE) = alone;
    }
}

// ------------------------------------------------------------------------------------------------
// k_cascade_rest: the lists of all layers, a layer's shared by its workgroups -- or, when the chain stopped at a dense layer (and wrote
// the lists before it), that layer and all after it on the tiles of k_cascade_fused.  Before those the assignments that the
// graph leaves open (META_ALONE; the chain wrote these layers' lists), on the same tiles.  Layer 0 is a step that inherits
// every token: Algorithm 1's step 5 on the identity list is Definition 2.2.
// A step is dealt as items, one per workgroup that its tiles can use.  A workgroup takes an item from the claim word of its
// XCD (step << 16 | items taken), from another XCD's when that is used up, and only then waits for the next step: whoever
// runs finishes the step, so the waits end however few workgroups are resident, and nothing is assumed about that.  The
// workgroup that finishes a step moves the claim words on, then the hand-over word (step << 15 | size of the set): a claim
// carries the step that it is good for, also if its workgroup came for the step before.  (One word for all claims and one
// for all sign-offs, every step cut for all workgroups, took 42 us per layer at T=2048, d=4096 and 36 us at T=512, d=768
// in fp32.)
struct RestParams {
    ChainParams c;             // layers c.s.first .. + c.s.L - 1, outputs
    FusedParams f;             // shape, threshold, workspace of sequence 0; the per-layer pointers are set in the kernel
    int spin_limit;
    int list_mode;             // how the sets are read back: LIST_PLAIN or LIST_COHERENT
};

template <typename In, bool WIDE, int KG, int DMA>
__global__ __launch_bounds__(256 * KG) void k_cascade_rest(RestParams rp) {
    extern __shared__ __align__(16) char lds[];
    using G = FusedGeom<KG, DMA>;
    __shared__ int s_step, s_item, s_items, s_word, s_last;
    FusedParams p = rp.f;
    p.steps = 1;
    const int T = p.T, first = rp.c.s.first, n_layers = rp.c.s.L;
    const int groups = p.groups > 1 ? p.groups : 1, g = (int)blockIdx.x % groups, worker = (int)blockIdx.x / groups;
    const int workers = p.groups > 1 ? p.wpg : p.grid;
    int32_t* meta = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(rp.c.s.meta) + (long long)g * p.ws_gs);
    const int start = meta[META_PROGRESS];
    const unsigned long long alone = *reinterpret_cast<const unsigned long long*>(meta + META_ALONE);
    if (start >= first + n_layers) {
        const ScreenUnit SU(T, rp.c.s.nch, rp.c.s.edge_cap);
        const int items = n_layers * (rp.c.assign ? 2 : 1), parts = max(workers / items, 1);
        for (int i = worker; i < items * parts; i += workers) {
            const int j = i % items, part = i / items, l = j < n_layers ? j : j - n_layers;
            if ((alone >> l) & 1ull) continue;
            if (j < n_layers) screen_lists(rp.c, SU, l, g, reinterpret_cast<int*>(lds), part, parts);
            else screen_assign(rp.c, SU, l, g, reinterpret_cast<int*>(lds), part, parts);
        }
        if (alone == 0ull) return;
    }
    p.hits = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(p.hits) + (long long)g * p.ws_gs);
    p.ticket = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(p.ticket) + (long long)g * p.ws_gs);
    if (p.first) p.first = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(p.first) + (long long)g * p.ws_gs);
    int32_t* idx0 = rp.c.idx + (long long)g * p.list_gs;
    int32_t* adds0 = rp.c.adds ? rp.c.adds + (long long)g * p.list_gs : nullptr;
    int32_t* rem0 = rp.c.removes ? rp.c.removes + (long long)g * p.list_gs : nullptr;
    int32_t* cnt0 = rp.c.counts + (long long)g * p.counts_gs;
    unsigned long long* ops0 = rp.c.ops + (long long)g * p.ops_gs;
    const int per_layer = rp.c.assign ? 2 : 1;                // steps of a layer: the set, and the assignment to it if wanted
    const int n_alone = __popcll(alone), steps = n_alone + (first + n_layers - start) * per_layer;
    auto layer_of = [&](int step) {                           // (the assignments left open come first)
        if (step >= n_alone) return start + (step - n_alone) / per_layer;
        unsigned long long m = alone;
        for (int k = 0; k < step; ++k) m &= m - 1ull;
        return first + __ffsll((long long)m) - 1;
    };
    // worker w of a problem is on XCD (w groups + g) % 8, one of nx: the ones with equal w % nx share a claim word
    const int low = groups & -groups, nx = 8 / (low < 8 ? low : 8);
    int32_t* claim = meta + META_REST_CLAIM;
    auto items_of = [&](int r, bool triangle) {               // workgroups that a step on a set of r can use
        if (groups > 1) return workers;
        const int n = ((int)fused_step_deal<In, WIDE, KG, DMA>(p, r, triangle, (unsigned)workers).tiles + 7) / 8 * 8;
        return min(max(n, 8), workers);                       // (a step that is refused still has to be finished)
    };
    auto share = [&](int n, int x) { return n > x ? (n - x + nx - 1) / nx : 0; };   // of n items those with index % nx == x
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) {
            const int home = worker % nx;
            int step, part = home, item = -1, items = 0, word = -1;
            // polls a word until its upper bits have come to `least`; -1: given up (not reached: see above)
            auto wait_for = [&](const int32_t* w, int shift, int least) {
                for (int n = 0; n < rp.spin_limit; ++n) {
                    const int v = __hip_atomic_load(w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((v >> shift) >= least) return v;
                    __builtin_amdgcn_s_sleep(2);
                }
                return -1;
            };
            for (;;) {
                const int from = part, v = atomicAdd(claim + 32 * from, 1);
                step = v >> 16;
                if (step >= steps) break;
                const int epoch = wait_for(meta + META_REST_EPOCH, 15, step);
                bool gone = epoch < 0;
                part = home;
                if (!gone) {
                    if ((epoch >> 15) > step) continue;       // (this claim came too late for its step)
                    // the set that the step works with: of an earlier launch, of the layer before, of the step before
                    const int i = layer_of(step);
                    word = step < n_alone ? cnt0[(size_t)i * 4] : step > n_alone ? epoch & 0x7FFF : i == 0 ? T : cnt0[(size_t)(i - 1) * 4];
                    items = items_of(word, step == n_alone && i == 0);
                    if ((v & 0xFFFF) < share(items, from)) { item = (v & 0xFFFF) * nx + from; break; }
                    int u[8], other = -1;                     // what is left of the step elsewhere
#pragma unroll
                    for (int x = 0; x < 8; ++x)
                        u[x] = __hip_atomic_load(claim + 32 * (x < nx ? x : home), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int x = 0; x < 8; ++x)
                        if (x < nx && (u[x] >> 16) == step && (u[x] & 0xFFFF) < share(items, x)) other = x;
                    if (other >= 0) part = other;
                    else gone = wait_for(claim + 32 * home, 16, step + 1) < 0;
                }
                if (gone) {
                    cnt0[(size_t)layer_of(step) * 4 + 3] = ADA_ERR_DEVICE;
                    step = steps;
                    break;
                }
            }
            s_step = step;
            s_item = item;
            s_items = items;
            s_word = word;
        }
        __syncthreads();
        const int step = s_step, local = s_item, items = s_items, r = s_word;
        if (step >= steps) break;                             // uniform
        const int i = layer_of(step);
        const size_t row = (size_t)i * (size_t)T;
        p.X = reinterpret_cast<const char*>(rp.c.s.X[i - first]) + (long long)g * p.x_gs;
        p.assign_mode = step < n_alone || (per_layer == 2 && ((step - n_alone) & 1));
        if (p.assign_mode) {
            p.list_mode = rp.list_mode;
            p.prev_idx = idx0 + row;
            p.assign = rp.c.assign + row;
            p.pos_out = rp.c.pos + row;
            p.counts = rp.c.info + (size_t)i * 8;
        } else {
            p.list_mode = i == 0 ? LIST_IDENTITY : rp.list_mode;
            p.prev_idx = idx0 + row - (i == 0 ? 0 : T);
            p.idx = idx0 + row;
            p.adds = i > 0 && adds0 ? adds0 + row : nullptr;
            p.removes = i > 0 && rem0 ? rem0 + row : nullptr;
            p.counts = cnt0 + (size_t)i * 4;
            p.gram_ops = ops0 + i;
        }
        const bool r_ok = r >= 1 && r <= T;
        if (r_ok) fused_step_tiles<In, WIDE, KG, DMA>(p, r, p.list_mode == LIST_IDENTITY, lds, (unsigned)local, (unsigned)items, (unsigned)workers);
        const int jq = min((int)threadIdx.x, T - 1);
        const int q0 = list_at(p, jq), qp0 = list_at(p, max(jq - 1, 0));
        drain_stores();
        __syncthreads();
        if (threadIdx.x == 0) {
            const int x = local % nx, parts = items < nx ? items : nx;
            s_last = atomicAdd(p.ticket + TICKET_XCD0 + 32 * x, 1) == share(items, x) - 1 && atomicAdd(p.ticket, 1) == parts - 1 ? 1 : 0;
        }
        __syncthreads();
        if (s_last) {                                         // uniform
            if (threadIdx.x == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            __syncthreads();
            int r_new = r;
            if (p.assign_mode) assign_finish<G::THREADS>(p, r, r_ok, q0, qp0);
            else r_new = fused_update<G::THREADS>(p, r, r_ok, q0, qp0, lds + G::META, reinterpret_cast<int*>(lds + G::OFF_SCAN));
            __syncthreads();
            if (threadIdx.x == 0) {
                for (int x = 0; x < nx; ++x)
                    __hip_atomic_store(claim + 32 * x, (step + 1) << 16, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                __hip_atomic_store(meta + META_REST_EPOCH, ((step + 1) << 15) | (r_new & 0x7FFF), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    // the last workgroup of the sequence to leave puts the counters back to zero
    if (threadIdx.x == 0 && atomicAdd(meta + META_REST_LEFT, 1) == workers - 1) {
        for (int x = 0; x < nx; ++x) __hip_atomic_store(claim + 32 * x, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(meta + META_REST_EPOCH, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(meta + META_REST_LEFT, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(meta + META_PROGRESS, first + n_layers, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

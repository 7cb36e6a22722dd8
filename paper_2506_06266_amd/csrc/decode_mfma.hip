// Serve-time decode over a shared cartridge (Sec. 3.3; decode step of Sec. 2.3) on the matrix
// cores, bf16, head_dim 128.  One query token per request; keys = [prefix Z ; the request's own
// KV], all visible.
//
// The cartridge is shared by every request, so its part is a real GEMM: the B*G query rows
// that read one KV head (G = Hq/Hkv) are stacked and run against the prefix, split along the
// prefix into workgroups of 128 rows (prefix role).  The ragged own-KV part is bandwidth-bound:
// the packed own caches are cut evenly along their token axis, whatever the requests' lengths,
// and every resident wavefront streams one range of one KV head through a private LDS slot, with
// the G query rows of the request it is passing padded into one 32-column MFMA block (own role).
// Both roles are workgroups of one launch (decode_fused_kernel), sized so that two share a CU --
// the matrix-core work on the L2-resident cartridge overlaps the HBM streaming of the own caches
// instead of preceding it -- and the launch holds no more workgroups than the chip keeps
// resident.  Every split writes a normalised partial (O, lse); decode_merge_kernel combines them
// by their log-sum-exps.
//
// Composition (Sec. 5.4: cartridges trained apart are concatenated without retraining) and the
// per-request cartridges of App. A.3's serving protocol use the same two kernels: the shared
// prefix is a list of segments, each split and run like a single cartridge (a segment is never
// copied next to another), and a request's private cartridge is streamed like its own KV.
#include <limits.h>
#include <math.h>

#include "attn_mfma.h"

namespace cart {
using namespace mfma;

constexpr int DEC_BM = 128;            // stacked query rows per prefix workgroup (4 x 32)
constexpr int DEC_BN = 32;             // prefix keys per LDS tile
#ifndef DEC_NBUF
#define DEC_NBUF 4                     // prefix tiles in LDS: one read, one ready, the rest in flight
#endif
constexpr int DEC_TILE_B = DEC_BN * ROW_B;
constexpr int DEC_SUB = 32;            // own keys per wavefront step
constexpr int DEC_SUB_B = DEC_SUB * ROW_B;

constexpr int DEC_MIN_SHARE = 64;       // fewest rows per streamed range of requests that are not shorter
constexpr int DEC_FINE_LEN = 512;       // longest request whose ranges may be of one step
constexpr int DEC_LEAN_SHARE = 256;     // the lean plans' (unless no request is that long)
constexpr int DEC_POOL_STEPS = 2;       // fewest steps per range beside private cartridges
constexpr int DEC_MAX_SPLIT = 48;       // most parts the shared prefix is split into
constexpr int DEC_MAX_PARTS = 64;       // most ranges the longest request's own rows are cut into
constexpr int DEC_FEW_ROWS = 2048;      // output rows up to which the merge takes four wavefronts a row
constexpr int DEC_MAX_SEG = CART_MAX_SEGMENTS;
constexpr size_t DEC_STATIC_BYTES = static_cast<size_t>(32) << 20;   // the library's own scratch array (cart_decode_static)

// The shared prefix as a list of segments (one for a single cartridge), by value in the kernel
// arguments.  Segment s is split along its slots into n_ps[s] parts of tiles_per_split[s] tiles;
// its workgroups are blockIdx [blk0[s], blk0[s+1]) and its partial results slots slot0[s] + part.
struct PrefixTable {
    const bf16_t* zk[DEC_MAX_SEG];
    const bf16_t* zv[DEC_MAX_SEG];
    int p[DEC_MAX_SEG], tiles_per_split[DEC_MAX_SEG], n_ps[DEC_MAX_SEG], slot0[DEC_MAX_SEG];
    int blk0[DEC_MAX_SEG + 1];
    int n_seg;
};

struct DecodePlan {
    PrefixTable tab;
    int G, n_rb, n_ps;                    // prefix: row blocks, partial slots of all segments
    // streamed rows (own tokens, then private cartridges): rows per range of either, most ranges one request's
    // own rows / private cartridge reach into, first range of the private cartridges, workgroups
    int share, pool_share, n_oc, n_cc, pool_r0, n_own_wg;
    size_t part_o_bytes, part_l_bytes;
};

// Tiles per part of one of several segments, where the estimate says tps: parts of one length, one part fewer where they are at most a
// quarter longer for it; where tps is at most 3, as few as a quarter takes, rounded up to whole tiles (one more than tps then).  By the
// estimate's length a segment of 64 tiles was 52 and 12.  us a call, by the estimate's length / so: 128 requests, 8192 slots in 4 segments 79.8 /
// 65.4; 4, 20116 in 4 26.9 / 21.4; 44, 18406 in 3 34.4 / 36.2; 206 drawn problems of 2 to 8 segments 1.05 times as fast, 0.95 at worst (as few parts as
// a quarter takes of any tps 1.04, 0.93; parts levelled and no longer 1.01, 0.94; none longer than tps where that is at most 3: 1.05, 0.95, few requests
// up to 0.09 slower: three requests, 995 slots in 3 11.0 / 12.0).
static int segment_tiles(int tiles, int tps) {
    if (tps <= 3) {
        const int parts = (4 * tiles + 5 * tps - 1) / (5 * tps);
        return (tiles + parts - 1) / parts;
    }
    const int parts = (tiles + tps - 1) / tps, fewer = parts > 1 ? (tiles + parts - 2) / (parts - 1) : tiles;
    return 4 * fewer <= 5 * tps ? fewer : (tiles + parts - 1) / parts;
}

// seg_p[n_seg]: slots per shared segment; pool_p: slots of a private cartridge (0 = none);
// T: rows of the packed own caches
// lean > 0: prefix workgroups for the chip and no more, and long ranges; 1: in no more parts than
// the estimate takes either.
static DecodePlan make_plan(int B, int Hq, int Hkv, int max_own_len, int T, const int* seg_p, int n_seg, int pool_p, int lean) {
    DecodePlan p;
    p.G = Hq / Hkv;
    const int rows = B * p.G;
    p.n_rb = (rows + DEC_BM - 1) / DEC_BM;
    int total_tiles = 0;
    for (int s = 0; s < n_seg; ++s) total_tiles += (seg_p[s] + DEC_BN - 1) / DEC_BN;
    // Into how many parts the prefix is split: the cheapest by an estimate of the fused kernel (the
    // longer of a prefix workgroup and a streaming wavefront) plus the partials' way to the merge.  A
    // prefix workgroup takes 8 us and 0.55 us per tile, 0.8 on a CU it shares; a stream 1.8 us per
    // step, or its bytes at 5.5 TB/s; a part of one output row 1 KB at 2 TB/s.  Measured, whole call
    // (us): 128 requests, 8192 shared slots, own rows U[1,1024]: 3 parts 83, 6 parts 75; with 2048
    // shared slots and a private cartridge of 2048 each: 6 parts 273, 3 parts 258, 1 part 252; 32
    // requests, 8192 slots: 24 parts 34.4, 12 parts 32.6; 128 requests of up to 100 own rows, 8192 slots: 6 parts, each workgroup
    // on a CU of its own, 35.3, more of them sharing CUs 42.1.
    const long stream_rows = pool_p > 0 ? static_cast<long>(T) + static_cast<long>(B) * pool_p : T;
    const float stream_us = static_cast<float>(stream_rows) * Hkv * 2 * ROW_B / 5.5e6f;
    const long chip = 2L * device_cus();          // workgroups the chip keeps resident (256 threads, two per CU)
    // steps of the own rows: a request takes at least one, half a step more than its rows on average
    const float own_steps = static_cast<float>(B) * fmaxf(static_cast<float>(T) / (static_cast<float>(B) * DEC_SUB) + 0.5f, 1.f);
    const float row_us = 2.5f * own_steps / static_cast<float>(T);       // of a wavefront's range, where it waits for memory
    // Rows per own range that leave every workgroup a CU of its own (0: none do, or the requests are so short that
    // such a range holds many of them: 205 requests of up to 10 own rows, 8 / 8 heads, 4103 slots 27.7 us a call, 32.3 so)
    auto unshared = [&](long n_pre) {
        const long room = chip / 2 - n_pre, ranges = room > 0 && (lean || T >= 16L * B) ? 4 * room / Hkv : 0;
        const long rows = ranges > 0 ? (static_cast<long>(T) + ranges - 1) / ranges : 0, to = rows < DEC_SUB ? 8 : DEC_SUB;
        return (rows + to - 1) / to * to;
    };
    int tps = 0;
    float tps_us = 0.f;
    for (int parts = 1; parts <= DEC_MAX_SPLIT && parts <= total_tiles; parts += 1 + parts / 8) {
        const int t = (total_tiles + parts - 1) / parts;
        const long n_pre = static_cast<long>(Hkv) * p.n_rb * parts;
        if (parts > 1 && n_pre > chip - 64) break;
        const long waves = 4 * (chip - n_pre < 64 ? 64 : chip - n_pre);
        const float steps = ceilf(static_cast<float>(stream_rows) * Hkv / (static_cast<float>(waves) * DEC_SUB));
        const float stream = fmaxf(4.f + 1.8f * steps, stream_us);
        float us = fmaxf(8.f + (stream_us > 20.f || (pool_p == 0 && T >= 16L * B) ? 0.8f : 0.55f) * static_cast<float>(t), stream);
        const long own = pool_p == 0 && stream_us <= 20.f ? unshared(n_pre) : 0;
        if (own > 0) us = fminf(us, fmaxf(8.f + 0.55f * static_cast<float>(t), 4.f + row_us * static_cast<float>(own)));
        us += static_cast<float>(parts) * B * Hq * 2 * HD * 4 / 2.0e6f;
        if (parts == 1 || us < tps_us) {
            tps_us = us;
            tps = t;
        }
    }
    if (lean && total_tiles > 0) {
        const int parts = (192 + Hkv * p.n_rb - 1) / (Hkv * p.n_rb), t = (total_tiles + parts - 1) / parts;
        tps = lean == 1 && t < tps ? tps : t;
    }
    p.tab.n_seg = 0;
    p.tab.blk0[0] = 0;
    p.n_ps = 0;
    int longest = tps;
    for (int s = 0; s < n_seg; ++s) {
        const int nPt = (seg_p[s] + DEC_BN - 1) / DEC_BN;
        if (nPt == 0) continue;                                     // an empty segment adds nothing
        const int k = p.tab.n_seg++;
        p.tab.p[k] = seg_p[s];
        p.tab.tiles_per_split[k] = nPt == total_tiles ? tps : segment_tiles(nPt, tps);
        longest = longest > p.tab.tiles_per_split[k] ? longest : p.tab.tiles_per_split[k];
        p.tab.n_ps[k] = (nPt + p.tab.tiles_per_split[k] - 1) / p.tab.tiles_per_split[k];
        p.tab.slot0[k] = p.n_ps;
        p.n_ps += p.tab.n_ps[k];
        p.tab.blk0[k + 1] = p.tab.blk0[k] + Hkv * p.n_rb * p.tab.n_ps[k];
        p.tab.zk[k] = p.tab.zv[k] = nullptr;                        // filled by the launcher
    }
    // Streamed rows: the workgroups that stay resident beside the prefix workgroups, four wavefronts
    // each, one wavefront per (range, KV head); the ranges cut the own rows of all requests, then the
    // private cartridges of all requests evenly, in whole steps of 32 rows where they are that long.
    const int n_pre_wg = p.n_ps > 0 ? p.tab.blk0[p.tab.n_seg] : 0;
    long wgs = chip - n_pre_wg;
    if (wgs < 64) wgs = 64;
    long ranges = 4 * wgs / Hkv;
    if (ranges < 1) { ranges = 1; wgs = (Hkv + 3) / 4; }
    // (not below DEC_MIN_SHARE rows, nor the longest request in more than DEC_MAX_PARTS ranges: shorter
    // ranges only multiply the partials a request leaves.  8 requests of up to 500 tokens, us a call:
    // at least 256 / 128 / 64 / 32 rows -> 23.0 / 18.7 / 17.9 / 17.8; one of 16000: 19 / 17.8 / 25.4 / 36.9.
    // A step each where every workgroup still has a CU of its own and no request leaves many partials: a launch of few
    // requests ends with its longest range, whose steps follow one another.  us from a graph, 64 rows -> 32: 4 requests of up
    // to 150 rows, 2048 slots 13.8 -> 11.8; 8 of up to 300, 8 / 2 heads, 4096 slots 14.0 -> 12.1; 16 of up to 150 15.7 -> 14.5;
    // but 99 of up to 134 without a cartridge, which then share CUs, 16.8 -> 19.0, 7 of up to 1930 12.7 -> 13.3.  Where the
    // ranges' ends fall in the requests moves one call by 10 % down and 18 % up; over 16 sets of lengths: 5 of up to 77 rows 1.06
    // times as fast, 9 of up to 79 1.05, 100 of up to 69, 8 / 2 heads, 1.04, 40 of up to 90 1.03, 53 of up to 321, 8 / 2, 1.00.
    // Requests shorter than that on average take a step each however few their rows are, so a range then
    // holds about one of them: 31 requests of up to 17 tokens beside 885 slots 26.2 -> 18.2, 128 of up to 16
    // beside 1000 33.6 -> 22.2, 48 of up to 53 beside 516 20.9 -> 18.2)
    auto up = [](long x, long to) { return (x + to - 1) / to * to; };
    const long least = (static_cast<long>(max_own_len) + DEC_MAX_PARTS - 1) / DEC_MAX_PARTS;
    long share, used;                                                        // rows per own range, ranges that hold rows
    p.pool_share = p.pool_r0 = p.n_cc = 0;
    if (pool_p == 0) {
        const long resident = (static_cast<long>(T) + ranges - 1) / ranges, needed = resident > least ? resident : least, avg = up(T / B, 8);
        share = up(needed, DEC_SUB);
        if (lean) {
            // (a range as long as the longest request takes no fewer partials: up to 256 rows were 256 steps where every
            // request had one: 404 requests, 28 / 4 heads, 3161 slots 549 us a call, 46 so)
            const long most = up(max_own_len, DEC_SUB);
            const long wanted = most < DEC_LEAN_SHARE ? most : DEC_LEAN_SHARE;
            share = share > wanted ? share : wanted;
        }
        else {
            const bool fine = max_own_len <= DEC_FINE_LEN && n_pre_wg + (((static_cast<long>(T) + share - 1) / share) * Hkv + 3) / 4 <= chip / 2;
            const long min_share = fine ? DEC_SUB : DEC_MIN_SHARE;
            if (avg < min_share) share = avg > needed ? avg : up(needed, needed < DEC_SUB ? 8 : DEC_SUB);
            else if (share < min_share) share = min_share;
        }
        if (share < 8) share = 8;
        used = (static_cast<long>(T) + share - 1) / share;
        // From the workgroup on that shares a CU the prefix role takes longer (the 0.55 and 0.8 us above): longer ranges
        // where they leave every workgroup its own CU and the launch ends sooner for it.  212 requests, 8 / 2 heads, 10891
        // slots, up to 184 own rows: ranges of 64 rows (360 workgroups) 38.5 us a call, of 192 (238) 31.6; 200 requests,
        // 4096 slots, up to 300 rows 28.1, now 26.2.  (By the longest part there is where that is longer than the estimate's: 22 such
        // problems 0.86 to 1.34 times as fast, 1.09 in the mean; by a shorter one 38 others 0.82 to 1.20, 0.98 in the mean.)
        const long longer = n_pre_wg > 0 ? unshared(n_pre_wg) : 0;
        if (longer > share) {
            const float tiles = static_cast<float>(longest);
            if (1.1f * fmaxf(8.f + 0.55f * tiles, 4.f + row_us * static_cast<float>(longer)) <=
                fmaxf(8.f + 0.8f * tiles, 4.f + row_us * static_cast<float>(share))) {
                share = longer;
                used = (static_cast<long>(T) + share - 1) / share;
            }
        }
    } else {
        // Beside private cartridges: by steps, so that a range of short requests (a step each) takes as long as
        // one of cartridge rows.  Cut by rows alone (us a call): 208 requests of up to 40 own rows, cartridges of 786
        // slots 230, now 179; 121 requests, cartridges of 389 265, now 70; 223 requests, cartridges of one slot 458, now 63.
        const float pool_steps = ceilf(static_cast<float>(pool_p) / DEC_SUB);
        const float each = fmaxf((own_steps + static_cast<float>(B) * pool_steps) / static_cast<float>(ranges > 4 ? ranges - 2 : ranges),
                                 static_cast<float>(DEC_POOL_STEPS));        // steps per range
        auto cut = [&](float x, long at_least) {
            const long r = static_cast<long>(x) > at_least ? static_cast<long>(x) : at_least;
            return up(r < 8 ? 8 : r, r <= DEC_SUB ? 8 : DEC_SUB);
        };
        share = cut(each * static_cast<float>(T) / own_steps, least);
        p.pool_share = static_cast<int>(cut(each * static_cast<float>(pool_p) / pool_steps, 0));
        p.pool_r0 = static_cast<int>((static_cast<long>(T) + share - 1) / share);
        used = p.pool_r0 + (static_cast<long>(B) * pool_p + p.pool_share - 1) / p.pool_share;
        p.n_cc = (pool_p + p.pool_share - 1) / p.pool_share + 1;
        wgs = (used * Hkv + 3) / 4;
    }
    if ((used * Hkv + 3) / 4 < wgs) wgs = (used * Hkv + 3) / 4;
    p.share = static_cast<int>(share);
    p.n_own_wg = static_cast<int>(wgs);
    p.n_oc = static_cast<int>((max_own_len + share - 1) / share) + 1;
    const size_t slots = static_cast<size_t>(p.n_ps + p.n_cc + p.n_oc) * B * Hq;
    p.part_o_bytes = (slots * HD * sizeof(float) + 255) & ~static_cast<size_t>(255);
    p.part_l_bytes = (slots * sizeof(float) + 255) & ~static_cast<size_t>(255);
    return p;
}
// A plan whose partials exceed the library's own scratch array gives way to a lean one that fits it, so that
// finer cuts never keep a problem from cart_decode_static (whose bits are cart_decode's); with private
// cartridges there is no such entry point.  The finer cut is no faster at those sizes (128 requests, 512 slots,
// 9000 own rows at most: 400 us either way; 96, 1000 slots, 12000: 393; 256, 2048, 3000: 85), but 208 requests of
// up to 40 own rows, 47 shared slots and cartridges of 786 lost 32 us of 262 to a lean plan.
DecodePlan decode_plan(int B, int Hq, int Hkv, int max_own_len, int T, const int* seg_p, int n_seg, int pool_p) {
    const DecodePlan p = make_plan(B, Hq, Hkv, max_own_len, T, seg_p, n_seg, pool_p, 0);
    if (pool_p == 0 && p.part_o_bytes + p.part_l_bytes > DEC_STATIC_BYTES)
        for (int lean = 1; lean <= 2; ++lean) {
            const DecodePlan l = make_plan(B, Hq, Hkv, max_own_len, T, seg_p, n_seg, 0, lean);
            if (l.part_o_bytes + l.part_l_bytes <= DEC_STATIC_BYTES) return l;
        }
    return p;
}

// Prefix role of the fused kernel: 128 stacked query rows (32 per wavefront) against one split of
// one segment, 32 keys per LDS tile, DEC_NBUF tiles in rotation.  Small on purpose -- at most 256 registers
// per lane and 64 KB of LDS -- so that two workgroups share a CU and the bandwidth-bound own-KV
// role runs beside it.  part_o [slot][B][Hq][128] fp32 (normalised), part_l [slot][B][Hq]
// (natural-log lse).
__device__ __forceinline__ void decode_prefix_role(char* sm, const bf16_t* __restrict__ q, const PrefixTable& tab,
                                                   float* __restrict__ part_o, float* __restrict__ part_l, int B,
                                                   int Hq, int Hkv, float c, int n_rb, int blk) {
    const int G = Hq / Hkv;
    int seg = 0;
    while (seg + 1 < tab.n_seg && blk >= tab.blk0[seg + 1]) ++seg;
    int id = blk - tab.blk0[seg];
    const int hk = id % Hkv; id /= Hkv;
    const int rb = id % n_rb;
    const int sp = id / n_rb;
    const bf16_t* zk = tab.zk[seg];
    const bf16_t* zv = tab.zv[seg];
    const int P = tab.p[seg], tiles_per_split = tab.tiles_per_split[seg];
    const int slot_base = tab.slot0[seg];
    const int lane = threadIdx.x & 63, lg = lane >> 5, lc = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rows = B * G;
    const int rho = rb * DEC_BM + 32 * wv + lc;

    bf16x8 qf[8];
    {
        const int rc = min(rho, rows - 1);
        const bf16_t* qp = q + (static_cast<size_t>(rc / G) * Hq + hk * G + rc % G) * HD + 8 * lg;
#pragma unroll
        for (int t = 0; t < 8; ++t) qf[t] = *reinterpret_cast<const bf16x8*>(qp + 16 * t);
    }
    const int nPt = (P + DEC_BN - 1) / DEC_BN;
    const int t_lo = sp * tiles_per_split;
    const int nT = min(tiles_per_split, nPt - t_lo);
    const char* zk_b = reinterpret_cast<const char*>(zk) + static_cast<size_t>(hk) * P * ROW_B;
    const char* zv_b = reinterpret_cast<const char*>(zv) + static_cast<size_t>(hk) * P * ROW_B;
    char* smk = sm;
    char* smv = sm + DEC_NBUF * DEC_TILE_B;
    auto issue = [&](int t, int buf) __attribute__((always_inline)) {   // 2 + 2 loads per wavefront
        const int j0 = (t_lo + t) * DEC_BN;
        tile_load_async<DEC_BN>(smk + buf * DEC_TILE_B, zk_b, j0, P - 1, ROW_B);
        tile_load_async<DEC_BN>(smv + buf * DEC_TILE_B, zv_b, j0, P - 1, ROW_B);
    };

    f32x16 acc[4];
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[db][r] = 0.f;
    float m_run = NEG_BIG, l_run = 0.f;
    f32x16 s;
    auto scores = [&](const char* kt) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
        for (int t8 = 0; t8 < 8; ++t8) s = mma(lds_frag_n(kt, lc, 16 * t8 + 8 * lg), qf[t8], s);
    };
    // entries past the last slot of the segment, in the scores of tile t
    auto mask_tail = [&](int t) __attribute__((always_inline)) {
        const int j0 = (t_lo + t) * DEC_BN;
        if (j0 + DEC_BN > P) {
            const int thr = P - 1 - j0 - 4 * lg;
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + (r & 3) > thr) s[r] = NEG_BIG;
        }
    };
    // largest scaled score of the tile in s, over both halves of the lane's row
    auto row_max = [&]() __attribute__((always_inline)) {
        float tm = s[0];
#pragma unroll
        for (int r = 1; r < 16; ++r) tm = fmaxf(tm, s[r]);
        return partner_max(tm) * c;
    };

    // Pipeline.  Entering iteration u a wavefront holds, in registers, the masked scores of tile
    // u, the K fragments of tile u+1 and the V fragments of tile u.  The iteration issues the 8
    // score products of tile u+1 and the 8 O products of tile u; each fragment register is
    // refilled from LDS right behind the product that consumed it (K of tile u+2, V of tile u+1),
    // and the exponentials of tile u run between the score products.  Requested all together
    // behind the barrier instead, the four wavefronts' 64 KB of fragment reads per tile keep LDS
    // busy for as long as the products keep the matrix cores busy, one after the other.
    //   What bounds an iteration is the number of instructions the one wavefront of a SIMD has to
    // issue besides its 16 products (measured 0.74 us per tile against 0.25 us of products with
    // about 250 of them), so everything that is not per-element work is kept out of the loop:
    //   - the loop is unrolled over the DEC_NBUF buffers, which makes every LDS address of an
    //     iteration a per-lane constant plus an immediate;
    //   - the softmax reference m is the maximum of the FIRST tile and is not looked for again:
    //     the exponentials are formed against it, and only if a lane's row sum for the tile
    //     exceeds 2^12 -- some score lies more than 2^8 above m, or the sum has overflowed -- does
    //     the wavefront take the tile's true maximum, rescale O and l, and form the tile's
    //     exponentials again.  A false alarm costs time, not accuracy.
    // Buffers: tiles u+1 and u+2 are read, tile u+3 is in flight, the buffer of tile u is free
    // once every wavefront's reads of it have completed -- the wait and the barrier at the top --
    // and takes tile u+4.  Past the end of the split the last tile is requested again and stale
    // buffers are read; nothing formed from them is used.
    static_assert(DEC_NBUF == 4, "the rotation below is written for four buffers");
    constexpr float OVER = 4096.f;
#pragma unroll
    for (int t = 0; t < DEC_NBUF; ++t) issue(min(t, nT - 1), t);
    dma_wait_but<4 * (DEC_NBUF - 2)>();          // tiles 0 and 1
    __syncthreads();
    scores(smk);
    mask_tail(0);
    m_run = row_max();
    bf16x8 ka[8], va[2][4];
#pragma unroll
    for (int t8 = 0; t8 < 8; ++t8) ka[t8] = lds_frag_n(smk + DEC_TILE_B, lc, 16 * t8 + 8 * lg);
#pragma unroll
    for (int db = 0; db < 4; ++db) {
        va[0][db] = lds_frag_t(smv, 0, 32 * db, lane);
        va[1][db] = lds_frag_t(smv, 16, 32 * db, lane);
    }
    auto body = [&](auto buf_c, int u) __attribute__((always_inline)) {
        constexpr int BUF = decltype(buf_c)::value;
        dma_wait_but<4 * (DEC_NBUF - 3)>();       // tile u+2
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __syncthreads();
        issue(min(u + DEC_NBUF, nT - 1), BUF);
        const char* kn = smk + ((BUF + 2) % DEC_NBUF) * DEC_TILE_B;
        const char* vn = smv + ((BUF + 1) % DEC_NBUF) * DEC_TILE_B;
        f32x16 sn;
        uint32_t pw[8];
        float rs = 0.f;
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t8 = 0; t8 < 8; ++t8) {
            // written out so that the product stays in this place: the compiler is free to move
            // the builtin across the fences, and gathers all eight at the end of the iteration.
            // sn is next read by vector instructions behind the eight O products.
            if (t8 == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(sn) : "v"(ka[0]), "v"(qf[0]));
            else         asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(sn) : "v"(ka[t8]), "v"(qf[t8]));
            ka[t8] = lds_frag_n(kn, lc, 16 * t8 + 8 * lg);
            const float p0 = fast_exp2(fmaf(s[2 * t8], c, -m_run));
            const float p1 = fast_exp2(fmaf(s[2 * t8 + 1], c, -m_run));
            rs += p0;
            rs += p1;
            pw[t8] = pack_bf16x2(p0, p1);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (__any(!(rs <= OVER))) {
            const float m_new = fmaxf(m_run, row_max());
            const float alpha = fast_exp2(m_run - m_new);
            l_run *= alpha;
            m_run = m_new;
#pragma unroll
            for (int db = 0; db < 4; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[db][r] *= alpha;
            rs = 0.f;
#pragma unroll
            for (int t8 = 0; t8 < 8; ++t8) {
                const float p0 = fast_exp2(fmaf(s[2 * t8], c, -m_run));
                const float p1 = fast_exp2(fmaf(s[2 * t8 + 1], c, -m_run));
                rs += p0 + p1;
                pw[t8] = pack_bf16x2(p0, p1);
            }
        }
        l_run += rs;
        const bf16x8 pf0 = __builtin_bit_cast(bf16x8, u32x4{pw[0], pw[1], pw[2], pw[3]});
        const bf16x8 pf1 = __builtin_bit_cast(bf16x8, u32x4{pw[4], pw[5], pw[6], pw[7]});
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int db = 0; db < 4; ++db) {
            acc[db] = mma(va[0][db], pf0, acc[db]);
            va[0][db] = lds_frag_t(vn, 0, 32 * db, lane);
            __builtin_amdgcn_sched_barrier(0);
            acc[db] = mma(va[1][db], pf1, acc[db]);
            va[1][db] = lds_frag_t(vn, 16, 32 * db, lane);
            __builtin_amdgcn_sched_barrier(0);
        }
        s = sn;
        if (u + 1 < nT) mask_tail(u + 1);
    };
    for (int u0 = 0; u0 < nT; u0 += DEC_NBUF) {
        body(std::integral_constant<int, 0>{}, u0);
        if (u0 + 1 < nT) body(std::integral_constant<int, 1>{}, u0 + 1);
        if (u0 + 2 < nT) body(std::integral_constant<int, 2>{}, u0 + 2);
        if (u0 + 3 < nT) body(std::integral_constant<int, 3>{}, u0 + 3);
    }
    dma_wait();
    const float l_tot = l_run + partner(l_run);
    const float inv = 1.f / l_tot;
    if (rho < rows) {
        const size_t slot = (static_cast<size_t>(slot_base + sp) * B + rho / G) * Hq + hk * G + rho % G;
        float* op = part_o + slot * HD;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                typedef float f32x4 __attribute__((ext_vector_type(4)));
                f32x4 w = {acc[db][4 * r4] * inv, acc[db][4 * r4 + 1] * inv, acc[db][4 * r4 + 2] * inv,
                           acc[db][4 * r4 + 3] * inv};
                *reinterpret_cast<f32x4*>(op + 32 * db + 8 * r4 + 4 * lg) = w;
            }
        if (lg == 0) part_l[slot] = (m_run + fast_log2(l_tot)) * CART_LN2;
    }
}

// One step of the own-KV role: 32 key rows (the last ones of a run repeated past its end and
// masked) from the wavefront's private 16 KB LDS slot against the G query rows of one request,
// which occupy columns 0..G-1 of one MFMA block.
struct OwnState {
    f32x16 acc[4];
    float m_run, l_run;
};
__device__ __forceinline__ void own_reset(OwnState& st) {
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) st.acc[db][r] = 0.f;
    st.m_run = NEG_BIG;
    st.l_run = 0.f;
}
// nkeys: valid keys of the step (1..32)
__device__ __forceinline__ void own_step(OwnState& st, const bf16x8 (&ka)[8], const bf16x8 (&va)[2][4],
                                         const bf16x8 (&qf)[8], int nkeys, float c, int lg) {
    f32x16 s;
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int t8 = 0; t8 < 8; ++t8) s = mma(ka[t8], qf[t8], s);
    if (nkeys < DEC_SUB) {
        const int thr = nkeys - 1 - 4 * lg;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (8 * (r >> 2) + (r & 3) > thr) s[r] = NEG_BIG;
    }
    float tm = s[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) tm = fmaxf(tm, s[r]);
    tm = partner_max(tm) * c;
    // the running maximum moves only when exceeded by more than RESCALE_GAP (then O and l are
    // rescaled; rare after a run's first step)
    const float m_new = tm > st.m_run + RESCALE_GAP ? tm : st.m_run;
    if (__any(m_new != st.m_run)) {
        const float alpha = fast_exp2(st.m_run - m_new);
        st.l_run *= alpha;
        st.m_run = m_new;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) st.acc[db][r] *= alpha;
    }
    float rs = 0.f;
    f32x16 p;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        p[r] = fast_exp2(fmaf(s[r], c, -st.m_run));
        rs += p[r];
    }
    st.l_run += rs;
    const bf16x8 pf0 = pack_frag(p, 0), pf1 = pack_frag(p, 8);
#pragma unroll
    for (int db = 0; db < 4; ++db) {
        st.acc[db] = mma(va[0][db], pf0, st.acc[db]);
        st.acc[db] = mma(va[1][db], pf1, st.acc[db]);
    }
}
// normalised partial O and natural-log lse of the G rows (lanes lc < G) into partial slot `slot`
__device__ __forceinline__ void own_store(const OwnState& st, float* __restrict__ part_o, float* __restrict__ part_l,
                                          size_t slot_row0, int G, int lc, int lg) {
    const float l_tot = st.l_run + partner(st.l_run);
    const float inv = 1.f / l_tot;
    if (lc < G) {
        const size_t slot = slot_row0 + lc;
        float* op = part_o + slot * HD;
#pragma unroll
        for (int db = 0; db < 4; ++db)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                typedef float f32x4 __attribute__((ext_vector_type(4)));
                f32x4 w = {st.acc[db][4 * r4] * inv, st.acc[db][4 * r4 + 1] * inv, st.acc[db][4 * r4 + 2] * inv,
                           st.acc[db][4 * r4 + 3] * inv};
                *reinterpret_cast<f32x4*>(op + 32 * db + 8 * r4 + 4 * lg) = w;
            }
        if (lg == 0) part_l[slot] = (st.m_run + fast_log2(l_tot)) * CART_LN2;
    }
}
// 32 rows x 256 B from row `row0` of a [rows][pitch] tensor (rows past `lim` repeat row lim) into
// the wavefront's slot: 8 direct-to-LDS loads of 4 rows each, per tensor
template <bool ONCE>
__device__ __forceinline__ void own_issue(const char* k_row0, const char* v_row0, uint32_t pitch, int lim, char* kt,
                                          char* vt, int lane) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int r = 4 * i + (lane >> 4);
        const uint32_t off = static_cast<uint32_t>(min(r, lim)) * pitch + (((lane & 15) ^ swz(r)) << 4);
        if constexpr (ONCE) {
            dma16_nt(k_row0, off, lds_addr(kt) + 4 * i * ROW_B);
            dma16_nt(v_row0, off, lds_addr(vt) + 4 * i * ROW_B);
        } else {
            dma16(k_row0, off, lds_addr(kt) + 4 * i * ROW_B);
            dma16(v_row0, off, lds_addr(vt) + 4 * i * ROW_B);
        }
    }
}
__device__ __forceinline__ void own_frags(const char* kt, const char* vt, bf16x8 (&ka)[8], bf16x8 (&va)[2][4], int lane) {
    const int lg = lane >> 5, lc = lane & 31;
#pragma unroll
    for (int t8 = 0; t8 < 8; ++t8) ka[t8] = lds_frag_n(kt, lc, 16 * t8 + 8 * lg);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int db = 0; db < 4; ++db) va[ks][db] = lds_frag_t(vt, 16 * ks, 32 * db, lane);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}
__device__ __forceinline__ void own_load_q(const bf16_t* __restrict__ q, int b, int Hq, int hk, int G, int lc, int lg,
                                           bf16x8 (&qf)[8]) {
    const bf16_t* qp = q + (static_cast<size_t>(b) * Hq + hk * G + min(lc, G - 1)) * HD + 8 * lg;
#pragma unroll
    for (int t = 0; t < 8; ++t) qf[t] = *reinterpret_cast<const bf16x8*>(qp + 16 * t);
}

// Own-KV role.  The own caches of all requests are one packed tensor [T][Hkv][128], so the work
// is cut evenly along T whatever the requests' lengths: wavefront (range r, KV head hk) streams
// token rows [r*share, (r+1)*share) of head hk, 32 rows per step, without a pause where one
// request ends and the next begins -- the next step's rows are requested before the current step
// is computed, and the next request's query rows are fetched while the current request runs.
// A step never spans two requests (its tail is masked), and every (request, range) pair leaves
// one partial: request b's slot j is range cu[b]/share + j.  Equal bytes per wavefront, all
// wavefronts resident from the start: nothing depends on the order or the pace at which the
// hardware hands out workgroups.  (One workgroup per four (request, head, chunk) items, left
// to the dispatcher, measured 20 us slower on the serving shape: by the middle of the kernel 50
// to 90 CUs sat empty with hundreds of workgroups still to start.)
template <bool ONCE>
__device__ __forceinline__ void decode_own_stream(char* sm, const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                  const bf16_t* __restrict__ v, const int32_t* __restrict__ cu,
                                                  float* __restrict__ part_o, float* __restrict__ part_l, int B, int Hq,
                                                  int Hkv, float c, int slot0, int n_oc, int share, int r, int hk) {
    const int G = Hq / Hkv;
    const int lane = threadIdx.x & 63, lg = lane >> 5, lc = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long t_lo_l = static_cast<long>(r) * share;
    // The request b the range starts in (cu[b] <= t_lo < cu[b+1]), its rows, the end of the next one and of all.  Up to 128
    // requests' offsets are two loads, a lane each, and the last one: a single trip to memory ahead of the first rows, not three.
    const int T = cu[B];
    int b, req_lo, req_hi, next_hi;
    if (B <= 128) {
        const int c0 = cu[min(lane, B)], c1 = cu[min(lane + 64, B)];
        if (t_lo_l >= T) return;
        const int t = static_cast<int>(t_lo_l);
        b = static_cast<int>(__popcll(__ballot(lane > 0 && lane <= B && c0 <= t)) + __popcll(__ballot(lane + 64 <= B && c1 <= t)));
        if (b >= B) return;                       // (cu not increasing: nothing sensible to do)
        auto at = [&](int i) __attribute__((always_inline)) {
            return i >= B ? T : i < 64 ? __builtin_amdgcn_readlane(c0, i) : __builtin_amdgcn_readlane(c1, i - 64);
        };
        req_lo = at(b);
        req_hi = at(b + 1);
        next_hi = at(b + 2);
    } else {
        if (t_lo_l >= T) return;
        int cnt = 0;
        for (int i = lane + 1; i <= B; i += 64) cnt += cu[i] <= static_cast<int>(t_lo_l) ? 1 : 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, CART_WAVE);
        b = __builtin_amdgcn_readfirstlane(cnt);
        if (b >= B) return;
        req_lo = cu[b];
        req_hi = cu[b + 1];
        next_hi = b + 2 <= B ? cu[b + 2] : T;
    }
    const int t_lo = static_cast<int>(t_lo_l), t_hi = min(t_lo + share, T);
    int run_end = min(req_hi, t_hi);          // rows [t, run_end) belong to request b
    const uint32_t pitch = static_cast<uint32_t>(Hkv) * ROW_B;
    const char* k_h = reinterpret_cast<const char*>(k) + static_cast<size_t>(hk) * ROW_B;
    const char* v_h = reinterpret_cast<const char*>(v) + static_cast<size_t>(hk) * ROW_B;
    char* kt = sm + (2 * wv) * DEC_SUB_B;
    char* vt = kt + DEC_SUB_B;
    bf16x8 qf[8], qn[8];
    own_load_q(q, b, Hq, hk, G, lc, lg, qf);
    own_load_q(q, min(b + 1, B - 1), Hq, hk, G, lc, lg, qn);
    OwnState st;
    own_reset(st);
    int t = t_lo;
    own_issue<ONCE>(k_h + static_cast<size_t>(t) * pitch, v_h + static_cast<size_t>(t) * pitch, pitch, run_end - 1 - t, kt, vt,
              lane);
    for (;;) {
        const int nkeys = min(DEC_SUB, run_end - t);
        const bool run_last = t + DEC_SUB >= run_end;
        const int t_next = run_last ? run_end : t + DEC_SUB;
        const bool more = t_next < t_hi;
        const int next_end = run_last ? min(next_hi, t_hi) : run_end;
        bf16x8 ka[8], va[2][4];
        dma_wait();                      // this step's rows have landed
        own_frags(kt, vt, ka, va, lane); // into registers; the slot then takes the next step's rows
        if (more)
            own_issue<ONCE>(k_h + static_cast<size_t>(t_next) * pitch, v_h + static_cast<size_t>(t_next) * pitch, pitch,
                      next_end - 1 - t_next, kt, vt, lane);
        own_step(st, ka, va, qf, nkeys, c, lg);
        if (run_last) {
            const int j = r - req_lo / share;
            if (j < n_oc)      // (always, unless a request is longer than the max_own_len the caller stated)
                own_store(st, part_o, part_l, (static_cast<size_t>(slot0 + j) * B + b) * Hq + hk * G, G, lc, lg);
            if (!more) break;
            ++b;
            req_lo = req_hi;
            req_hi = next_hi;
            run_end = next_end;
            next_hi = b + 2 <= B ? cu[b + 2] : T;
#pragma unroll
            for (int i = 0; i < 8; ++i) qf[i] = qn[i];
            own_load_q(q, min(b + 1, B - 1), Hq, hk, G, lc, lg, qn);
            own_reset(st);
        }
        t = t_next;
    }
}

// The private cartridges pool[cart_id[b]] ([Hkv,pool_p,128]; none for a request whose cart_id is
// negative), streamed like own rows, as rows b * pool_p ...: a wavefront's range r may cross from one
// cartridge to the next, and every (request, range) pair leaves one partial.  (Chunks of a cartridge dealt out round-robin left
// wavefronts with two chunks beside others with one: 128 cartridges of 2048 slots beside 2048
// shared ones took 371 us a call against 273, and 252 with the prefix in one part.)
__device__ __forceinline__ void decode_pool_stream(char* sm, const bf16_t* __restrict__ q,
                                                   const bf16_t* __restrict__ pool_k, const bf16_t* __restrict__ pool_v,
                                                   const int32_t* __restrict__ cart_id, int pool_p,
                                                   float* __restrict__ part_o, float* __restrict__ part_l, int B, int Hq,
                                                   int Hkv, float c, int slot0, int share, int once_from, int r, int hk) {
    const int G = Hq / Hkv;
    const int lane = threadIdx.x & 63, lg = lane >> 5, lc = lane & 31;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long lo = static_cast<long>(r) * share;                   // positions among the cartridges' rows: [lo, hi)
    const long hi = min(lo + share, static_cast<long>(B) * pool_p);
    if (lo >= hi) return;
    char* kt = sm + (2 * wv) * DEC_SUB_B;
    char* vt = kt + DEC_SUB_B;
    // the rows of the first request from b on that has a cartridge: slots [s, end) of it
    struct Run { int b, s, end; bool once; const char *k, *v; };
    auto run_from = [&](int b, int s) __attribute__((always_inline)) {
        Run w = {-1, 0, 0, false, nullptr, nullptr};
        for (; b < B && static_cast<long>(b) * pool_p + s < hi; ++b, s = 0) {
            const int cid = cart_id ? cart_id[b] : -1;
            if (cid < 0) continue;
            const size_t off = (static_cast<size_t>(cid) * Hkv + hk) * pool_p * ROW_B;
            w.b = b;
            w.s = s;
            w.end = static_cast<int>(min(static_cast<long>(pool_p), hi - static_cast<long>(b) * pool_p));
            w.k = reinterpret_cast<const char*>(pool_k) + off;
            w.v = reinterpret_cast<const char*>(pool_v) + off;
            break;
        }
        return w;
    };
    // whether a cartridge is no other request's and its rows are not kept in the caches (see DEC_ONCE_BYTES)
    auto read_once = [&](int b) __attribute__((always_inline)) {
        const int cid = cart_id[b];
        int same = 0, with = 0;
        for (int i0 = 0; i0 < B; i0 += 4 * CART_WAVE) {
            int id[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) id[j] = cart_id[min(i0 + j * CART_WAVE + lane, B - 1)];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const bool is = i0 + j * CART_WAVE + lane < B;
                same += static_cast<int>(__popcll(__ballot(is && id[j] == cid)));
                with += static_cast<int>(__popcll(__ballot(is && id[j] >= 0)));
            }
        }
        return same == 1 && with >= once_from;
    };
    const int b0 = static_cast<int>(lo / pool_p);
    Run cur = run_from(b0, static_cast<int>(lo - static_cast<long>(b0) * pool_p));
    if (cur.b < 0) return;
    bf16x8 qf[8];
    OwnState st;
    // (the range's first rows ahead of what says who else reads them)
    own_issue<false>(cur.k + static_cast<size_t>(cur.s) * ROW_B, cur.v + static_cast<size_t>(cur.s) * ROW_B, ROW_B, cur.end - 1 - cur.s, kt, vt, lane);
    const bool may = once_from <= B;    // (the other requests' numbers: on their way together with rows that have been requested)
    if (may) cur.once = read_once(cur.b);
    while (cur.b >= 0) {
        own_load_q(q, cur.b, Hq, hk, G, lc, lg, qf);
        own_reset(st);
        Run nxt = run_from(cur.b + 1, 0);
        if (may && nxt.b >= 0) nxt.once = read_once(nxt.b);
        for (int s = cur.s; s < cur.end; s += DEC_SUB) {
            bf16x8 ka[8], va[2][4];
            dma_wait();
            own_frags(kt, vt, ka, va, lane);
            const bool last = s + DEC_SUB >= cur.end;
            const char* kn = last ? nxt.k : cur.k;
            const char* vn = last ? nxt.v : cur.v;
            const int sn = last ? nxt.s : s + DEC_SUB, en = last ? nxt.end : cur.end;
            const bool once = last ? nxt.once : cur.once;
            if (kn) {
                kn += static_cast<size_t>(sn) * ROW_B;
                vn += static_cast<size_t>(sn) * ROW_B;
                if (once) own_issue<true>(kn, vn, ROW_B, en - 1 - sn, kt, vt, lane);
                else      own_issue<false>(kn, vn, ROW_B, en - 1 - sn, kt, vt, lane);
            }
            own_step(st, ka, va, qf, min(DEC_SUB, cur.end - s), c, lg);
        }
        const int j = r - static_cast<int>(static_cast<long>(cur.b) * pool_p / share);
        own_store(st, part_o, part_l, (static_cast<size_t>(slot0 + j) * B + cur.b) * Hq + hk * G, G, lc, lg);
        cur = nxt;
    }
}

// Both roles in one launch, two workgroups per CU: prefix workgroups (matrix-core and LDS work
// on data that sits in L2) and own-KV workgroups (HBM streaming) alternate in the grid while
// both kinds remain, so that the two run side by side instead of one after the other.  The
// launch holds no more workgroups than the chip keeps resident.
// ONCE: the own rows are not kept in the caches; pool_once: from how many requests with a cartridge on those are not that only one of them
// has (see DEC_ONCE_BYTES)
template <bool ONCE>
__global__ __launch_bounds__(256, 2) void decode_fused_kernel(
    const bf16_t* __restrict__ q, const PrefixTable tab, const bf16_t* __restrict__ k,
    const bf16_t* __restrict__ v, const int32_t* __restrict__ cu, const bf16_t* __restrict__ pool_k,
    const bf16_t* __restrict__ pool_v, const int32_t* __restrict__ cart_id, int pool_p,
    int pool_r0, int pool_share, int pool_once, float* __restrict__ part_o, float* __restrict__ part_l, int B, int Hq, int Hkv, float c,
    int n_rb, int n_cc, int n_oc, int share, int n_ps, int n_pre_wg, int n_own_wg) {
    constexpr int pre_b = 2 * DEC_NBUF * DEC_TILE_B, own_b = 4 * 2 * DEC_SUB_B;   // the two roles share one LDS block
    __shared__ __attribute__((aligned(16))) char sm[pre_b > own_b ? pre_b : own_b];
    const int i = blockIdx.x;
    const int both = min(n_pre_wg, n_own_wg);
    bool pre;
    int idx;
    // The roles alternate in runs of 8 workgroups (consecutive workgroups go to the 8 XCDs in
    // turn): every XCD hosts both roles, and with 8 KV heads a prefix workgroup's head
    // (idx % Hkv) is its XCD, whose L2 then holds that one head's cartridge.
    const int both8 = both & ~7;
    if (i < 2 * both8) { pre = !((i >> 3) & 1); idx = ((i >> 4) << 3) | (i & 7); }
    else               { const int r = i - 2 * both8, left = both - both8;
                         if (r < 2 * left) { pre = !(r & 1); idx = both8 + (r >> 1); }
                         else              { pre = n_pre_wg > n_own_wg; idx = i - both; } }
    if (pre) {
        decode_prefix_role(sm, q, tab, part_o, part_l, B, Hq, Hkv, c, n_rb, idx);
        return;
    }
    // every wavefront on its own from here on: no barrier in this role
    const int wid = __builtin_amdgcn_readfirstlane(idx * 4 + static_cast<int>(threadIdx.x >> 6));
    const int r = wid / Hkv, hk = wid - r * Hkv;
    if (n_cc > 0 && r >= pool_r0)
        decode_pool_stream(sm, q, pool_k, pool_v, cart_id, pool_p, part_o, part_l, B, Hq, Hkv, c, n_ps, pool_share, pool_once, r - pool_r0, hk);
    else
        decode_own_stream<ONCE>(sm, q, k, v, cu, part_o, part_l, B, Hq, Hkv, c, n_ps + n_cc, n_oc, share, r, hk);
}

// o[b,h,:] = sum_i w_i part_o[i] / sum_i w_i, w_i = exp(lse_i - max lse), over the partial slots
// that exist for the request: the n_ps prefix parts, one per range of `pool_share` rows its private
// cartridge (when it has one) and of `share` rows its own rows reach into.  WPR wavefronts per (b, h): one where there
// are rows for the whole chip, four where there are not (one request of 16000 own tokens: 19.9 -> 17.4
// us a call; 8 of up to 16000: 59.0 -> 54.0; above DEC_FEW_ROWS 4096 rows: 75 -> 81).  Slots in
// groups of 64: lane i holds the lse and the weight of the group's slot i, then every lane accumulates
// its two head elements over the wavefront's share of the group, eight slots' loads in flight.
template <int WPR>
__global__ __launch_bounds__(256) void decode_merge_kernel(const float* __restrict__ part_o,
                                                           const float* __restrict__ part_l,
                                                           const int32_t* __restrict__ cu,
                                                           const int32_t* __restrict__ cart_id, int pool_p, int pool_share,
                                                           bf16_t* __restrict__ o,
                                                           float* __restrict__ lse, int B, int Hq,
                                                           int n_ps, int n_cc, int n_oc, int share) {
    __shared__ float2 sub_sum[4][64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, sub = wv % WPR;
    const long row = static_cast<long>(blockIdx.x) * (4 / WPR) + wv / WPR;
    if (row >= static_cast<long>(B) * Hq) return;       // (WPR = 4: the whole workgroup)
    const int n = n_ps + n_cc + n_oc;
    const size_t stride = static_cast<size_t>(B) * Hq;
    // With few rows a launch is its round trips to memory: the wavefront's first eight slots are requested ahead of what says
    // which slots exist and what they weigh (us a call: four requests of up to 150 rows, 2048 shared slots 11.95 -> 11.59; one of up to
    // 3548 beside two cartridges 13.6 -> 12.8).  With rows for the whole chip the slots that do not exist cost more than the trip (128
    // requests, 8192 slots 72.0 -> 72.8).
    constexpr bool AHEAD = WPR == 4;
    float2 x[8];
    float first_l = 0.f;
    auto load8_any = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 8; ++j) x[j] = *reinterpret_cast<const float2*>(part_o + (min(i0 + j, n - 1) * stride + row) * HD + 2 * lane);
    };
    if constexpr (AHEAD) {
        load8_any(8 * sub);
        first_l = part_l[min(lane, n - 1) * stride + row];
    }
    const int b = row / Hq;
    int priv = 0;
    if (n_cc > 0 && cart_id && cart_id[b] >= 0) {
        const long p0 = static_cast<long>(b) * pool_p;
        priv = static_cast<int>((p0 + pool_p - 1) / pool_share - p0 / pool_share) + 1;
    }
    const int own = min(n_oc, (cu[b + 1] - 1) / share - cu[b] / share + 1);
    auto valid = [&](int i) { return i < n && (i < n_ps || (i < n_ps + n_cc ? i - n_ps < priv : i - n_ps - n_cc < own)); };
    auto slot_l = [&](int i) { return AHEAD && i < 64 ? first_l : part_l[i * stride + row]; };
    // slots in groups of 64: lane i holds the lse and the weight of slot g0 + i
    float m = -3.0e38f;
    for (int g0 = 0; g0 < n; g0 += 64)
        if (valid(g0 + lane)) m = fmaxf(m, slot_l(g0 + lane));
    m = wave_max(m);
    float wsum = 0.f, a0 = 0.f, a1 = 0.f;
    for (int g0 = 0; g0 < n; g0 += 64) {
        const int cnt = min(64, n - g0);
        const float wi = valid(g0 + lane) ? __expf(slot_l(g0 + lane) - m) : 0.f;
        wsum += wi;
        for (int i = 8 * sub; i < cnt; i += 8 * WPR) {
            if constexpr (!AHEAD) {
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    x[j] = float2{0.f, 0.f};
                    if (valid(g0 + i + j)) x[j] = *reinterpret_cast<const float2*>(part_o + ((g0 + i + j) * stride + row) * HD + 2 * lane);
                }
            } else if (g0 > 0 || i > 8 * sub) {
                load8_any(g0 + i);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float w = __shfl(wi, (i + j) & 63);
                const bool ok = !AHEAD || valid(g0 + i + j);       // (what a slot that does not exist holds may be anything)
                a0 = fmaf(w, ok ? x[j].x : 0.f, a0);
                a1 = fmaf(w, ok ? x[j].y : 0.f, a1);
            }
        }
    }
    if constexpr (WPR == 4) {
        sub_sum[wv][lane] = float2{a0, a1};
        __syncthreads();
        if (wv != 0) return;
#pragma unroll
        for (int w = 1; w < 4; ++w) {
            a0 += sub_sum[w][lane].x;
            a1 += sub_sum[w][lane].y;
        }
    }
    wsum = wave_sum(wsum);
    const float inv = 1.f / wsum;
    *reinterpret_cast<uint32_t*>(o + row * HD + 2 * lane) = pack_bf16x2(a0 * inv, a1 * inv);
    if (lane == 0 && lse) lse[row] = m + __logf(wsum);
}

// What the workspace queries return: the plan's bytes, or more, so that a workspace kept for a server's
// largest step serves its smaller ones (which are cut further): the most a cut of this problem or a smaller
// one can take, up to the size of the static array.  (A problem beyond that is asked for as it is.)
static size_t workspace_bytes(const DecodePlan& p, int B, int Hq, int max_own_len, const int* seg_p, int n_seg, int pool_p) {
    long tiles = 0;
    for (int s = 0; s < n_seg; ++s) tiles += (seg_p[s] + DEC_BN - 1) / DEC_BN;
    const long own = (static_cast<long>(max_own_len) + 7) / 8;
    const long slots = (tiles < DEC_MAX_SPLIT + n_seg ? tiles : DEC_MAX_SPLIT + n_seg) + (own < DEC_MAX_PARTS ? own : DEC_MAX_PARTS) + 1 +
                       (pool_p > 0 ? pool_p / DEC_SUB + 2 : 0);
    const size_t most = static_cast<size_t>(slots) * B * Hq * (HD + 1) * sizeof(float) + 512, bytes = p.part_o_bytes + p.part_l_bytes;
    const size_t kept = most < DEC_STATIC_BYTES ? most : DEC_STATIC_BYTES;
    return bytes > kept ? bytes : kept;
}

bool decode_mfma_supported(const cart_decode_desc& d) {
    return d.dtype == CART_BF16 && d.D == 128 && d.Hq / d.Hkv <= 32;
}

size_t decode_mfma_workspace(const cart_decode_desc& d) {
    const int n_seg = d.P > 0 ? 1 : 0;
    return workspace_bytes(decode_plan(d.B, d.Hq, d.Hkv, d.max_own_len, d.total_own_tokens, &d.P, n_seg, 0), d.B, d.Hq, d.max_own_len,
                           &d.P, n_seg, 0);
}

bool decode_composed_supported(const cart_decode_composed_desc& d) {
    return d.dtype == CART_BF16 && d.D == 128 && d.Hq / d.Hkv <= 32;
}

static DecodePlan composed_plan(const cart_decode_composed_desc& d, const cart_segment* shared) {
    int seg_p[DEC_MAX_SEG];
    for (int s = 0; s < d.n_shared; ++s) seg_p[s] = shared[s].p;
    return decode_plan(d.B, d.Hq, d.Hkv, d.max_own_len, d.total_own_tokens, seg_p, d.n_shared,
                     d.n_pool > 0 ? d.pool_p : 0);
}

size_t decode_composed_workspace(const cart_decode_composed_desc& d, const cart_segment* shared) {
    int seg_p[DEC_MAX_SEG];
    for (int s = 0; s < d.n_shared; ++s) seg_p[s] = shared[s].p;
    return workspace_bytes(composed_plan(d, shared), d.B, d.Hq, d.max_own_len, seg_p, d.n_shared, d.n_pool > 0 ? d.pool_p : 0);
}

// Streamed rows are read once a step.  Kept in the caches all the same, they drive out what a later call or kernel could
// still find there, and past a size each other: us a call, kept / not, 32 requests, 32 / 8 heads, 1024 shared slots, by the
// MB of their own rows (columns: two or four such calls on rows of their own in turn; one behind 512 MB of other traffic):
//     64   23.3 / 25.4   25.4 / 26.0   29.1 / 28.2        160   41.6 / 37.8   42.6 / 38.2   44.6 / 40.6
//     96   26.5 / 29.2   31.8 / 29.7   33.8 / 32.0        192   48.1 / 41.7   48.2 / 42.4   49.8 / 45.0
//    128   32.7 / 33.8   37.7 / 34.6   39.6 / 36.9        384   82.5 / 71.6   82.6 / 72.3   82.7 / 74.0
// Two calls' rows fit in the 256 MB that the memory side caches up to about the line.  (It spares a program that loops over the same rows; one
// whose layers each have their own, the last column, could do without them in the caches from 64 MB on: up to 7 %.)  Own rows are judged by themselves
// (together with cartridges, of which the host knows only how many there may be, 16 requests with 96 MB of own rows and two cartridges of 4 MB 28.0 /
// 30.5; with one each, 65 MB, 36.1 / 34.7), cartridges by those that the requests name, beside own rows that are kept: only the device knows how many there
// are and which of them several requests read.  Those are kept (us a call, all kept / none / as here; 128 requests, 2048 shared slots, cartridges of 2048: 4 of 256 for all of
// them 97.9 / 146.2 / 89.0; 32 161.7 / 183.8 / 161.1; 64 179.8 / 188.5 / 179.5; one each 210.1 / 190.5 / 187.6, beside own rows of 242 MB
// 249.2 / 225.9 / 226.2; for one request in twenty, beside them 130.4 / 122.7 / 113.0).
constexpr size_t DEC_ONCE_BYTES = static_cast<size_t>(144) << 20;
static long once_rows(int Hkv) { return static_cast<long>(DEC_ONCE_BYTES / (static_cast<size_t>(Hkv) * 2 * ROW_B)); }   // rows kept at most
// prefix parts + private-cartridge chunks + own ranges (one launch), then the merge
static int run_decode(const DecodePlan& p, bool once, int pool_once, int B, int Hq, int Hkv, float scale, const void* q, const void* pool_k,
                      const void* pool_v, const int32_t* cart_id, int pool_p, const void* k, const void* v,
                      const int32_t* cu, void* o, float* lse, void* ws, hipStream_t st) {
    float* part_o = static_cast<float*>(ws);
    float* part_l = reinterpret_cast<float*>(static_cast<char*>(ws) + p.part_o_bytes);
    const float c = scale * CART_LOG2E;
    const bf16_t *Q = static_cast<const bf16_t*>(q), *K = static_cast<const bf16_t*>(k), *V = static_cast<const bf16_t*>(v),
                 *PK = static_cast<const bf16_t*>(pool_k), *PV = static_cast<const bf16_t*>(pool_v);
    trace_begin(st);   // kernel order: prefix + own (one launch), merge
    const int n_pre_wg = p.n_ps > 0 ? p.tab.blk0[p.tab.n_seg] : 0;
    auto fused = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(n_pre_wg + p.n_own_wg)), dim3(256), 0, st, Q,
                           p.tab, K, V, cu, PK, PV, cart_id, pool_p, p.pool_r0, p.pool_share, pool_once, part_o, part_l, B, Hq, Hkv, c, p.n_rb,
                           p.n_cc, p.n_oc, p.share, p.n_ps, n_pre_wg, p.n_own_wg);
    };
    if (once) fused(decode_fused_kernel<true>);
    else      fused(decode_fused_kernel<false>);
    trace_mark(st);
    const long rows = static_cast<long>(B) * Hq;
    auto merge = [&](auto kernel, int rows_per_wg) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((rows + rows_per_wg - 1) / rows_per_wg)), dim3(256), 0, st, part_o,
                           part_l, cu, cart_id, pool_p, p.pool_share, static_cast<bf16_t*>(o), lse, B, Hq, p.n_ps, p.n_cc, p.n_oc,
                           p.share);
    };
    if (rows <= DEC_FEW_ROWS) merge(decode_merge_kernel<4>, 1);
    else                      merge(decode_merge_kernel<1>, 4);
    trace_mark(st);
    return static_cast<int>(hipGetLastError());
}

int launch_decode_mfma(const cart_decode_desc& d, float scale, const void* q, const void* zk,
                       const void* zv, const void* k, const void* v, const int32_t* cu, void* o,
                       float* lse, void* ws, hipStream_t st) {
    DecodePlan p = decode_plan(d.B, d.Hq, d.Hkv, d.max_own_len, d.total_own_tokens, &d.P, d.P > 0 ? 1 : 0, 0);
    if (p.tab.n_seg > 0) {
        p.tab.zk[0] = static_cast<const bf16_t*>(zk);
        p.tab.zv[0] = static_cast<const bf16_t*>(zv);
    }
    return run_decode(p, d.total_own_tokens > once_rows(d.Hkv), INT_MAX, d.B, d.Hq, d.Hkv, scale, q, nullptr, nullptr, nullptr, 0, k, v, cu, o,
                      lse, ws, st);
}

// ---- the decode step for callers that cannot allocate ---------------------------------------------
// The partial results of one call live in a file-scope device array instead of a caller-supplied
// workspace.  Each GPU holds its own copy of the array at its own address, looked up once per
// device; host code only ever uses that looked-up address, never the array's name.
static __device__ __align__(256) unsigned char scratch[DEC_STATIC_BYTES];
constexpr int DEC_MAX_DEVICES = 64;
static void* g_scratch_ptr[DEC_MAX_DEVICES];      // per device, nullptr until looked up

size_t decode_static_capacity() { return DEC_STATIC_BYTES; }

// the current device's copy of the array (nullptr when the runtime refuses the lookup)
void* decode_static_scratch() {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= DEC_MAX_DEVICES) return nullptr;
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return nullptr;
        g_scratch_ptr[dev] = ptr;
    }
    return g_scratch_ptr[dev];
}

int launch_decode_composed(const cart_decode_composed_desc& d, float scale, const void* q,
                           const cart_segment* shared, const void* pool_k, const void* pool_v,
                           const int32_t* cart_id, const void* k, const void* v, const int32_t* cu, void* o,
                           float* lse, void* ws, hipStream_t st) {
    DecodePlan p = composed_plan(d, shared);
    int kseg = 0;
    for (int s = 0; s < d.n_shared; ++s) {
        if (shared[s].p <= 0) continue;
        p.tab.zk[kseg] = static_cast<const bf16_t*>(shared[s].z_k);
        p.tab.zv[kseg] = static_cast<const bf16_t*>(shared[s].z_v);
        ++kseg;
    }
    const bool pool = d.n_pool > 0 && d.pool_p > 0;
    const long kept = once_rows(d.Hkv);
    const bool once = d.total_own_tokens > kept;
    // (a wavefront looks at 256 requests' numbers at a time, hidden behind two steps of a cartridge: us a call, kept / looked at, 1000 requests, cartridges
    // of 256 slots 342 / 317, 300 of 130 67.9 / 60.2, but 2000 of 64 586 / 780, of 32 419 / 833)
    const bool look = pool && d.pool_p >= (d.B + 4 * CART_WAVE - 1) / (4 * CART_WAVE) * 2 * DEC_SUB;
    const int pool_once = look ? static_cast<int>((kept - (once ? 0 : d.total_own_tokens)) / d.pool_p + 1) : INT_MAX;
    return run_decode(p, once, pool_once, d.B, d.Hq, d.Hkv, scale, q, pool ? pool_k : nullptr, pool ? pool_v : nullptr, pool ? cart_id : nullptr,
                      pool ? d.pool_p : 0, k, v, cu, o, lse, ws, st);
}

}  // namespace cart

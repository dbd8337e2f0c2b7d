// ----------------------------------------------------------------------------
// Route engine: round-robin graphs of at most 1024 traffic links, 32 input
// ports per node and 4 lines per cycle and link.  One workgroup per scenario,
// thread i owns traffic link i: its FIFO, the injection stream that starts
// there and the arbitration for the lines entering it.
//
// Source routing.  A line carries its remaining route as one word: per hop
// the index of the next link among its node's traffic links (rt_bits bits,
// all ones: the line leaves the network), then, when some line has
// predecessors, its flow.  The link's own lanes follow each other, so the
// next lane is a lane constant plus the low bits and no path table is read.
//
// Requests.  The k-th offered line of a FIFO goes to the post slot (k, input
// port) of the node it stands at, and its port bit into word k of the target
// lane: the target finds the first min(b, free) requests in round-robin order
// (k, port after the pointer) by bit operations alone and reads just those
// posts.  Its own stream's offers stay in registers.
//
// A cycle of a scenario whose links move one line per cycle has two phases,
// each ended by a barrier that waits on LDS only:
//   R  last cycle's result: the clock, the departed head; then the requests;
//   G  targets grant and append (a single grant always departs); lines at
//      their last hop complete.
// With more lines per cycle a third phase decides the departures:
//   G  targets grant, append and write the grant bits of the sources;
//   D  sources depart their longest granted prefix; a grant behind a refused
//      line (void) is reported to its target, which keeps only the lines that
//      departed at the start of the next R (rare).
// Bound: the instructions, LDS round trips and barriers of one simulated
// cycle (all waves of a scenario share four SIMDs).  Counters: 190
// instructions per wave and cycle with one line per cycle (k = 8 fat-tree, 12
// waves, 532 quad-cycles per cycle), 357 on 8 domains of 8 behind a fabric
// (two lines per cycle, 10 waves, 1180 quad-cycles, 57 % of them waiting).
// Measured per processed cycle, against the engine that ran it before:
//   k = 8 fat-tree all-to-all, 768 links        0.88 us  (grid engine 3.07)
//   k = 4, 512 scenarios, b in {1, 2, 4}        2.2 us   (lane engine 7.3)
//   8 x 8 hierarchical all-reduce, 640 links    1.96 us  (lane engine 3.78)
// Rings in device memory with predecessors and four lines (engine_route<4,
// true, true>): the loop needs more than the 128 registers of 16 waves per
// compute unit, and keeps 8 vector registers in scratch.  With two cached
// descriptors instead of eight it keeps none: k = 4 fat-tree trees 6.4 -> 5.1
// ms, but all-pairs exchanges on meshes of 9 to 20, whose ranges wait on 8 to
// 19 flows, take 1 to 8 % longer; a rule between the two is not made yet.
// Picking and reading every granted post before the first append (instead of
// one after the other under a branch) made the last two 8-10 % slower: most
// cycles grant one line per link.
// ----------------------------------------------------------------------------
#include <hip/hip_runtime.h>

#include <type_traits>

#include "engine_common.h"

namespace simgpu {

namespace {

using namespace dev;

typedef uint32_t Quad __attribute__((ext_vector_type(4)));

constexpr int kPc = 8;  // predecessor descriptors of a range kept in registers

// index of the lowest set bit (all ones if there is none)
__device__ __forceinline__ uint32_t ctz32(uint32_t v) { return (uint32_t)(__ffs((int)v) - 1); }

// A scenario's cycles, unrolled to BM lines per link and cycle (BM >= the
// scenario's largest bandwidth).  HBM: FIFO rings in device memory, the
// entries that a cycle may need read one cycle ahead; else in LDS.
template <int BM, bool HBM, bool PREDS>
__device__ __forceinline__ void route_cycles(const DevNet &d, unsigned char *smem) {
    uint32_t *word = reinterpret_cast<uint32_t *>(smem + d.rt_off[0]);   // [BM][nl] request port masks
    uint2 *post = reinterpret_cast<uint2 *>(smem + d.rt_off[1]);         // [BM][np] {line, route from the target on}
    uint32_t *gr = reinterpret_cast<uint32_t *>(smem + d.rt_off[2]);     // [np] granted offers (BM == 1: cycle tag)
    uint32_t *gv = reinterpret_cast<uint32_t *>(smem + d.rt_off[3]);     // [np] BM > 1: void offers of the last cycle
    uint32_t *deliv = reinterpret_cast<uint32_t *>(smem + d.rt_off[4]);  // PREDS: [nflows]
    // 0: tag of the last cycle in which a line moved, 1: lines completed,
    // 2: earliest event of an idle cycle, 3: tag of the last cycle with voids
    uint32_t *red = reinterpret_cast<uint32_t *>(smem + d.rt_off[5]);
    uint2 *rxc = reinterpret_cast<uint2 *>(smem + d.rt_off[6]);          // !HBM: rings {line, route}
    uint32_t *rrd = reinterpret_cast<uint32_t *>(smem + d.rt_off[7]);    // !HBM: rings' ready cycles
    const int s = blockIdx.x;
    const int i = threadIdx.x;
    const int nl = d.nl;
    const int np = d.rt_np;
    unsigned char *hring = reinterpret_cast<unsigned char *>(d.gfifo + (size_t)s * d.fifo_total);
    const bool on = i < nl;
    const uint32_t rbits = (uint32_t)d.rt_bits, rsink = (1u << rbits) - 1u;

    // lane constants
    int link = 0;
    uint32_t b = 0, L = 1, cap = 0, P = 1, pbit = 0, pslot = 0, tin = 0, obase = 0, fbase = 0, fmask = 0;
    int R = 0, rend = 0;
    if (on) {
        link = d.ln_link[i];
        const size_t pi = (size_t)s * d.m + link;
        b = (uint32_t)d.bw[pi];
        L = (uint32_t)d.lat[pi];
        cap = (uint32_t)d.cap[pi];
        P = (uint32_t)d.ln_P[i];
        pbit = 1u << d.ln_port[i];
        pslot = (uint32_t)d.rt_pslot[i];
        tin = (uint32_t)d.rt_tin[i];
        obase = (uint32_t)d.rt_obase[i];
        fbase = (uint32_t)d.ln_fifo[i];
        fmask = (uint32_t)d.ln_mask[i];
        R = d.ln_srbeg[i];
        rend = d.ln_srend[i];
    }
    const uint32_t pmask = P >= 32u ? ~0u : (1u << P) - 1u;

    // the stream's current range, and the next one read ahead
    uint32_t c_start = 0, c_len = 0, c_code = 0, n_start = 0, n_len = 0, n_code = 0;
    int c_pd0 = 0, c_pd1 = 0, n_pd0 = 0, n_pd1 = 0;
    uint32_t o = 0;
    int32_t pf[PREDS ? kPc : 1];
    uint32_t pb[PREDS ? kPc : 1];
    // PREDS: lines of the current range known to be released; the
    // predecessor that holds back the next one
    uint32_t lim = 0, hf = 0, hb = 0;
    auto read_next = [&]() {
        if (R + 1 < rend) {
            n_start = d.r_start[R + 1];
            n_len = d.r_len[R + 1];
            n_code = d.rt_code[R + 1];
            if constexpr (PREDS) {
                n_pd0 = d.r_pd[R + 1];
                n_pd1 = d.r_pd[R + 2];
            }
        }
    };
    auto read_preds = [&]() {
        if constexpr (PREDS) {
#pragma unroll
            for (int q = 0; q < kPc; q++) {
                // (an absent descriptor reads the first one and is ignored)
                const uint32_t at = c_pd0 + q < c_pd1 ? (uint32_t)(c_pd0 + q) : 0u;
                pf[q] = d.pd_flow[at];
                pb[q] = d.pd_base[at];
            }
            lim = 0;
            hf = (uint32_t)pf[0];
            hb = pb[0];
            if (c_pd0 == c_pd1) lim = 0xFFFFFFFFu;
        }
    };
    if (R < rend) {
        c_start = d.r_start[R];
        c_len = d.r_len[R];
        c_code = d.rt_code[R];
        if constexpr (PREDS) {
            c_pd0 = d.r_pd[R];
            c_pd1 = d.r_pd[R + 1];
        }
        read_preds();
        read_next();
    }
    // lines of a range released by a predecessor whose flow has delivered v
    const bool whole = d.pd_omask == 0u;
    auto allow = [&](uint32_t v, uint32_t base) -> uint32_t {
        return v > base ? (whole ? 0xFFFFFFFFu : v - base) : 0u;
    };
    // Lines of the current range released from o on, at most n (n >= 1).  The
    // predecessor that held the stream back last is looked at first; every
    // other one is read only once it has let go.
    auto released_from = [&](uint32_t n) -> uint32_t {
        if constexpr (PREDS) {
            if (lim < o + n) {
                if (allow(deliv[hf], hb) <= o) return lim > o ? lim - o : 0u;
                uint32_t a = 0xFFFFFFFFu;
#pragma unroll
                for (int q = 0; q < kPc; q++) {
                    uint32_t v = allow(deliv[pf[q]], pb[q]);
                    v = c_pd0 + q < c_pd1 ? v : 0xFFFFFFFFu;
                    hf = v < a ? (uint32_t)pf[q] : hf;
                    hb = v < a ? pb[q] : hb;
                    a = v < a ? v : a;
                }
                for (int q = c_pd0 + kPc; q < c_pd1; q++) {
                    const uint32_t f = (uint32_t)d.pd_flow[q], bs = d.pd_base[q];
                    const uint32_t v = allow(deliv[f], bs);
                    hf = v < a ? f : hf;
                    hb = v < a ? bs : hb;
                    a = v < a ? v : a;
                }
                lim = a;
            }
            const uint32_t left = lim > o ? lim - o : 0u;
            return left < n ? left : n;
        } else {
            return n;
        }
    };
    // Move on by n lines.  Ranges hold at least one line each.  The loads of a
    // range change are drained here, so that no cycle waits for them (the
    // memory counter would make it wait for its own stores too).
    auto advance = [&](uint32_t n) {
        o += n;
        if (o >= c_len) {
            while (R < rend && o >= c_len) {
                o -= c_len;
                R++;
                if (R < rend) {
                    c_start = n_start;
                    c_len = n_len;
                    c_code = n_code;
                    c_pd0 = n_pd0;
                    c_pd1 = n_pd1;
                    read_preds();
                    read_next();
                }
            }
            __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        }
    };

    uint32_t *comp = d.completion + (size_t)s * d.T;
    const uint32_t Tu = (uint32_t)d.T;
    uint32_t t = 0, tag = 0;
    uint64_t processed = 0;
    int32_t state = d.T > 0 ? kRunRunning : kRunOk;
    uint32_t head = 0, occ = 0, rr = 0;  // ring position of the head; entries held
    uint32_t tx = 0, busy = 0;
    bool wvoid = false;  // this FIFO's void offers are marked in gv

    struct Ent { uint32_t x, c, y; };
    Ent e[BM];   // the first entries (k < occ)
#pragma unroll
    for (int k = 0; k < BM; k++) e[k] = Ent{0u, 0u, 0u};
    auto ring_quad = [&](uint32_t pos) -> Quad {
        const uint32_t q = fbase + (pos & fmask);
        if constexpr (HBM) {
            return *reinterpret_cast<const Quad *>(hring + q * 16u);
        } else {
            const uint2 v = rxc[q];
            return Quad{v.x, v.y, rrd[q], 0u};
        }
    };
    auto ring_get = [&](uint32_t pos) -> Ent {
        const Quad v = ring_quad(pos);
        return Ent{v.x, v.y, v.z};
    };
    auto ring_put = [&](uint32_t pos, const Ent &v) {
        const uint32_t q = fbase + (pos & fmask);
        if constexpr (HBM) {
            *reinterpret_cast<uint4 *>(hring + q * 16u) = make_uint4(v.x, v.c, v.y, 0u);
        } else {
            rxc[q] = make_uint2(v.x, v.c);
            rrd[q] = v.y;
        }
    };

    while (state == kRunRunning) {
        tag++;
        // ------------------------------------------------------------ R
        uint32_t nf = 0, ejm = 0, next = kNever;
        Quad nq[BM];  // entries BM .. 2 BM - 1 of the FIFO as the cycle starts (HBM or BM == 1)
        Ent ap[BM];  // entries appended this cycle
        if constexpr (HBM || BM == 1) {  // (read first: they are needed once the heads have left)
#pragma unroll
            for (int k = 0; k < BM; k++)
                if (((uint32_t)(BM + k) < occ) & (e[k].y <= t)) nq[k] = ring_quad(head + (uint32_t)(BM + k));
        }
        if (occ != 0u) {
            if constexpr (BM == 1) {
                const uint32_t h = e[0].c & rsink;
                const bool rdy = e[0].y <= t;
                next = rdy ? kNever : e[0].y;
                nf = rdy ? 1u : 0u;
                ejm = (rdy & (h == rsink)) ? 1u : 0u;
                if (rdy & (h != rsink)) {
                    post[pslot] = make_uint2(e[0].x, e[0].c >> rbits);
                    atomicOr(&word[obase + h], pbit);
                }
            } else {
                bool open = true;
#pragma unroll
                for (int k = 0; k < BM; k++) {
                    open = open & ((uint32_t)k < b) & ((uint32_t)k < occ);
                    if (open) {
                        if (e[k].y > t) {
                            next = e[k].y;
                            open = false;
                        } else {
                            const uint32_t h = e[k].c & rsink;
                            if (h == rsink) {
                                ejm |= 1u << k;
                            } else {
                                post[k * np + (int)pslot] = make_uint2(e[k].x, e[k].c >> rbits);
                                atomicOr(&word[k * nl + (int)(obase + h)], pbit);
                            }
                            nf++;
                        }
                    }
                }
            }
        }
        uint32_t ns = 0;          // lines the stream offers
        uint32_t sx[BM], sc[BM];  // (BM > 1: they may run into the next ranges)
        if (R < rend) {
            ns = released_from(b < c_len - o ? b : c_len - o);
#pragma unroll
            for (int k = 0; k < BM; k++) {
                sx[k] = c_start + o + (uint32_t)k;
                sc[k] = c_code;
            }
            if constexpr (BM > 1) {
                if ((ns == c_len - o) & (ns < b)) {
                    for (int q = R + 1; q < rend && ns < b; q++) {
                        const uint32_t st = d.r_start[q], len = d.r_len[q], code = d.rt_code[q];
                        uint32_t n = len < b - ns ? len : b - ns;
                        if constexpr (PREDS)
                            for (int z = d.r_pd[q]; z < d.r_pd[q + 1]; z++) {
                                const uint32_t a = allow(deliv[d.pd_flow[z]], d.pd_base[z]);
                                n = a < n ? a : n;
                            }
#pragma unroll
                        for (int k = 0; k < BM; k++)
                            if (((uint32_t)k >= ns) & ((uint32_t)k < ns + n)) {
                                sx[k] = st + (uint32_t)k - ns;
                                sc[k] = code;
                            }
                        ns += n;
                        if (n < len) break;
                    }
                }
            }
        }
        lds_fence_block();
        // ------------------------------------------------------------ G
        if (i == 0) red[2] = kNever;
        if (wvoid) {  // read by every target before the last barrier
            gv[pslot] = 0u;
            wvoid = false;
        }
        uint32_t g = 0, sgr = 0, lastp = 0;
        uint32_t gp[BM];  // granted (k << 8 | port) by rank
        uint32_t w[BM], any = 0;
#pragma unroll
        for (int k = 0; k < BM; k++) {
            w[k] = on ? word[k * nl + i] : 0u;
            any |= w[k];
        }
        if constexpr (HBM) {
            // the entries read in R arrive here, before this phase's stores are
            // issued (the memory counter counts both, in order)
#pragma unroll
            for (int k = 0; k < BM; k++) asm volatile("" : "+v"(nq[k]));
        }
        if (on) {
            if ((any | ns) != 0u) {
                uint32_t tot = 0;
#pragma unroll
                for (int k = 0; k < BM; k++) {
                    if (any != 0u) word[k * nl + i] = 0u;
                    w[k] |= (uint32_t)k < ns ? 1u << (P - 1u) : 0u;
                    if constexpr (BM > 1) tot += (uint32_t)__builtin_popcount(w[k]);
                }
                if constexpr (BM == 1) tot = 1u;
                const uint32_t room = cap - occ;
                g = b < room ? b : room;
                g = g < tot ? g : tot;
                const uint32_t ready = t + L;
                if constexpr (BM > 1) {  // bit 0 = the port at the pointer
#pragma unroll
                    for (int k = 0; k < BM; k++)
                        w[k] = rr == 0u ? w[k] : ((w[k] >> rr) | (w[k] << (P - rr))) & pmask;
                }
#pragma unroll
                for (int r = 0; r < BM; r++) {
                    if ((uint32_t)r < g) {  // (a wave stops at its largest count)
                        uint32_t p, kk = 0;
                        if constexpr (BM == 1) {
                            const uint32_t hi = w[0] & (~0u << rr);
                            p = ctz32(hi != 0u ? hi : w[0]);
                        } else {
                            uint32_t v = w[0];
#pragma unroll
                            for (int k = 1; k < BM; k++) {
                                const bool z = v == 0u;
                                kk = z ? (uint32_t)k : kk;
                                v = z ? w[k] : v;
                            }
                            const uint32_t low = v & (0u - v);
#pragma unroll
                            for (int k = 0; k < BM; k++) w[k] ^= kk == (uint32_t)k ? low : 0u;
                            p = ctz32(v) + rr;
                            p = p >= P ? p - P : p;
                        }
                        gp[r] = (kk << 8) | p;
                        lastp = p;
                        Ent v;
                        v.y = ready;
                        if ((p == P - 1u) & (kk < ns)) {  // the injection port
                            sgr++;
                            v.x = sx[0];
                            v.c = sc[0];
#pragma unroll
                            for (int k = 1; k < BM; k++) {
                                v.x = kk == (uint32_t)k ? sx[k] : v.x;
                                v.c = kk == (uint32_t)k ? sc[k] : v.c;
                            }
                        } else {
                            const uint2 q = post[(int)(kk * (uint32_t)np + tin + p)];
                            v.x = q.x;
                            v.c = q.y;
                            if constexpr (BM == 1) gr[tin + p] = tag;
                            else atomicOr(&gr[tin + p], 1u << kk);
                        }
                        ap[r] = v;
                        ring_put(head + occ + (uint32_t)r, v);
                    }
                }
            }
        }
        // a line at its last hop completes (BM == 1: here, as a grant always
        // departs and nothing reads the delivered counts in this phase)
        auto complete = [&](const Ent &v) {
            if (v.x < Tu) comp[v.x] = t + 1u;
            if constexpr (PREDS) atomicAdd(&deliv[v.c >> rbits], 1u);
        };
        uint32_t dep = 0;  // lines that leave this FIFO
        if constexpr (BM == 1) {
            if (ejm) complete(e[0]);
            const unsigned long long mv = __ballot((g != 0u) | (ejm != 0u)), me = __ballot(ejm != 0u);
            if ((i & 63) == 0) {
                if (mv != 0ull) red[0] = tag;
                if (me != 0ull) atomicAdd(&red[1], (uint32_t)__builtin_popcountll(me));
            }
            lds_fence_block();
            dep = nf != 0u ? (ejm != 0u ? 1u : (gr[pslot] == tag ? 1u : 0u)) : 0u;
        } else {
            lds_fence_block();
            // -------------------------------------------------------- D
            uint32_t ej = 0;
            if (nf != 0u) {
                const uint32_t gm = gr[pslot];
                if (gm != 0u) gr[pslot] = 0u;
                const uint32_t ok = gm | ejm;
                dep = ctz32(~ok);
                const uint32_t out = (1u << dep) - 1u;
                const uint32_t vd = gm & ~out;
                ej = ejm & out;
                if (vd != 0u) {
                    gv[pslot] = vd;
                    wvoid = true;
                }
#pragma unroll
                for (int k = 0; k < BM; k++)
                    if ((ej >> k) & 1u) complete(e[k]);
            }
            const unsigned long long mv = __ballot((dep | sgr) != 0u), md = __ballot(wvoid);
            uint32_t ne = 0;
#pragma unroll
            for (int k = 0; k < BM; k++) ne += (uint32_t)__builtin_popcountll(__ballot((ej >> k) & 1u));
            if ((i & 63) == 0) {
                if (mv != 0ull) red[0] = tag;
                if (md != 0ull) red[3] = tag;
                if (ne != 0u) atomicAdd(&red[1], ne);
            }
            if constexpr (!HBM) {  // the heads of the next cycle (this lane's own appends included)
#pragma unroll
                for (int k = 0; k < BM; k++) e[k] = ring_get(head + dep + (uint32_t)k);
            }
            lds_fence_block();
        }
        // ------------------------------------------------------------ state
        Ent nx[BM];
#pragma unroll
        for (int k = 0; k < BM; k++) nx[k] = Ent{nq[k].x, nq[k].y, nq[k].z};
        const bool moved = red[0] == tag;
        const uint32_t done = red[1];
        uint32_t cnt = g;
        bool reload = false;
        if constexpr (BM > 1) {
            if (red[3] == tag && g != 0u) {
                // some grants were void: keep the lines that departed
                uint32_t keep = 0;
#pragma unroll
                for (int r = 0; r < BM; r++) {
                    if ((uint32_t)r < g) {
                        const uint32_t p = gp[r] & 255u, kk = gp[r] >> 8;
                        const bool own = (p == P - 1u) & (kk < ns);
                        const uint32_t m = own ? 0u : gv[tin + p];
                        if ((m >> kk) & 1u) {
                            reload = true;
                        } else {
                            if (reload) ring_put(head + occ + keep, ap[r]);
                            lastp = p;
                            keep++;
                        }
                    }
                }
                cnt = keep;
            }
        }
        if (cnt != 0u) {
            tx += cnt;
            busy++;
            rr = lastp + 1u == P ? 0u : lastp + 1u;
        }
        if constexpr (BM == 1) {
            // the head: kept, the entry behind it, or the line just appended
            if (dep != 0u) e[0] = occ >= 2u ? nx[0] : ap[0];
            else if (occ == 0u) e[0] = ap[0];
        } else if constexpr (HBM) {
            if (!reload) {
                Ent ne[BM];
#pragma unroll
                for (int k = 0; k < BM; k++) {
                    ne[k] = e[k];
#pragma unroll
                    for (int q = 1; q <= BM; q++) {  // entry k + q of the cycle's start
                        const Ent &v = k + q < BM ? e[k + q < BM ? k + q : 0] : nx[k + q >= BM ? k + q - BM : 0];
                        const bool is = dep == (uint32_t)q;
                        ne[k].x = is ? v.x : ne[k].x;
                        ne[k].c = is ? v.c : ne[k].c;
                        ne[k].y = is ? v.y : ne[k].y;
                    }
                    const uint32_t a = dep + (uint32_t)k - occ;  // index among the appended lines
#pragma unroll
                    for (int q = 0; q < BM; q++) {
                        const bool is = a == (uint32_t)q;
                        ne[k].x = is ? ap[q].x : ne[k].x;
                        ne[k].c = is ? ap[q].c : ne[k].c;
                        ne[k].y = is ? ap[q].y : ne[k].y;
                    }
                }
#pragma unroll
                for (int k = 0; k < BM; k++) e[k] = ne[k];
            }
        }
        head += dep;
        occ += cnt - dep;
        if constexpr (BM > 1) {
            if (reload) {
#pragma unroll
                for (int k = 0; k < BM; k++) e[k] = ring_get(head + (uint32_t)k);
            }
        }
        if (sgr != 0u) advance(sgr);
        processed++;
        if (done == Tu) {
            state = kRunOk;
        } else if (moved) {
            t = t + 1u;
        } else {  // idle: the earliest ready time of a FIFO head
            uint32_t v = next;
#pragma unroll
            for (int sh = 32; sh >= 1; sh >>= 1) {
                const uint32_t u = (uint32_t)__shfl_xor((int)v, sh);
                v = u < v ? u : v;
            }
            if ((i & 63) == 0 && v != kNever) atomicMin(&red[2], v);
            lds_fence_block();
            v = red[2];
            if (v == kNever) state = kRunDeadlock;
            else t = v;
        }
        if (state == kRunRunning && (uint64_t)t > d.max_cycles) state = kRunMaxCycles;
        if (state == kRunRunning && processed > d.watchdog) state = kRunWatchdog;
    }
    if (on) {
        const size_t pi = (size_t)s * d.m + link;
        d.tx_lines[pi] = tx;
        d.busy[pi] = busy;
    }
    if (i == 0) {
        d.makespan[s] = d.T > 0 ? t + 1u : 0u;
        d.status[s] = state;
        d.cycles[s] = processed;
    }
}

template <int BM, bool HBM, bool PREDS>
__global__ void __launch_bounds__(1024) engine_route(DevNet d) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int s = blockIdx.x;
    const int i = threadIdx.x;
    const int nthr = blockDim.x;
    for (int j = i; j < d.rt_zero; j += nthr) reinterpret_cast<uint32_t *>(smem)[j] = 0u;
    // links without traffic report zero counters
    for (int j = i; j < d.m; j += nthr)
        if (d.link_lane[j] < 0) {
            d.tx_lines[(size_t)s * d.m + j] = 0;
            d.busy[(size_t)s * d.m + j] = 0;
        }
    lds_fence_block();
    // a scenario runs the loop of its own largest bandwidth
    uint32_t *red = reinterpret_cast<uint32_t *>(smem + d.rt_off[5]);
    if constexpr (BM > 1) {
        if (i < d.nl) atomicMax(&red[4], (uint32_t)d.bw[(size_t)s * d.m + d.ln_link[i]]);
        lds_fence_block();
    }
    const uint32_t sb = BM > 1 ? red[4] : 1u;
    if (sb <= 1u) {
        route_cycles<1, HBM, PREDS>(d, smem);
    } else if constexpr (BM >= 2) {
        if (sb <= 2u || BM == 2) route_cycles<2, HBM, PREDS>(d, smem);
        else if constexpr (BM >= 4) route_cycles<4, HBM, PREDS>(d, smem);
    }
}

template <int BM, bool HBM>
hipError_t launch_route2(const DevNet &d, hipStream_t st) {
    auto k = d.has_preds ? engine_route<BM, HBM, true> : engine_route<BM, HBM, false>;
    if (d.lds_bytes > 65536)
        (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, d.lds_bytes);
    hipLaunchKernelGGL(k, dim3((unsigned)d.S), dim3((unsigned)d.lane_threads), (unsigned)d.lds_bytes, st, d);
    return hipGetLastError();
}

template <int BM>
hipError_t launch_route1(const DevNet &d, hipStream_t st) {
    return d.engine == kEngineRouteHbm ? launch_route2<BM, true>(d, st) : launch_route2<BM, false>(d, st);
}

}  // namespace

hipError_t launch_route(const DevNet &d, hipStream_t st) {
    switch (d.bm) {
    case 1: return launch_route1<1>(d, st);
    case 2: return launch_route1<2>(d, st);
    default: return launch_route1<4>(d, st);
    }
}

}  // namespace simgpu

// HIP kernels of the simulator step and its adjoint, written for gfx950
// (wave64).  A lane group of 8 to 64 lanes owns one (scenario, link) segment
// or one (scenario, node).  Nothing here is a dense contraction, so there is
// no MFMA: the step is bound by chains of dependent loads and instructions.
//
// Floating point: agent positions are float and follow one fixed operation
// order (no contraction: the library is built with -ffp-contract=off), so the
// integer decisions they feed (arrival, vacancy, detector crossings) are
// reproducible; utilities, Gumbel noise, token buckets and departure
// accumulators are double.
#include "sim_internal.h"

#include <math.h>

#include <mutex>

namespace sim {

// ---------------------------------------------------------------------------
// helpers
// ---------------------------------------------------------------------------

// Workgroups are dispatched round-robin over the 8 XCDs; remap the block id
// so that each XCD walks one contiguous range of work (its L2 then holds
// neighbouring segments).  Bijective on [0, nblocks).
__device__ __forceinline__ int xcd_block()
{
    const int nb = gridDim.x, b = blockIdx.x;
    const int x = b & 7, k = b >> 3, q = nb >> 3, r = nb & 7;
    return x * q + (x < r ? x : r) + k;
}

// Same mapping for block b of a role that owns nb consecutive blocks whose
// first block id is a multiple of 8 (so b % 8 is still the XCD).
__device__ __forceinline__ int xcd_remap(int b, int nb)
{
    const int x = b & 7, k = b >> 3, q = nb >> 3, r = nb & 7;
    return x * q + (x < r ? x : r) + k;
}

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Scenario of work item `item` when items are numbered scenario-major, n per
// scenario: a scalar branch skips the integer division (tens of instructions
// per lane) in the common single-scenario case.
__device__ __forceinline__ int scenario_of(int item, int n, int S)
{
    if (S == 1) return 0;
    return item / n;
}

__device__ __forceinline__ double wave_sum_d(double v)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// One near-tie record (scenario, step, class, agent, link, decision), links
// in the internal numbering (the host maps them back).  Replays carry no log.
__device__ __forceinline__ void tie_record(const Dev &d, int s, int t, int cls, int ag, int link, int dec)
{
    if (!d.tie_log) return;
    const int k = atomicAdd(d.tie_n, 1);
    if (k >= d.tie_cap) return;
    int32_t *r = d.tie_log + 6 * (int64_t)k;
    r[0] = s; r[1] = t; r[2] = cls; r[3] = ag; r[4] = link; r[5] = dec;
}

// Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11): ten rounds of two
// 32x32->64 multiplies with the Weyl key schedule.
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        // one 32x32->64 product gives both halves (a single v_mad_u64_u32)
        const uint64_t p0 = (uint64_t)0xD2511F53u * c[0], p1 = (uint64_t)0xCD9E8D57u * c[2];
        const uint32_t lo0 = (uint32_t)p0, hi0 = (uint32_t)(p0 >> 32);
        const uint32_t lo1 = (uint32_t)p1, hi1 = (uint32_t)(p1 >> 32);
        const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
        c[0] = n0; c[1] = lo1; c[2] = n2; c[3] = lo0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// counter (agent, step, purpose + 2*block, 0); purpose 0 = link choice with
// one word per candidate, 1 = merge (word 0)
__device__ __forceinline__ void draw4(uint64_t seed, int agent, int step, int purpose, int block, uint32_t w[4])
{
    w[0] = (uint32_t)agent; w[1] = (uint32_t)step; w[2] = (uint32_t)(purpose + 2 * block); w[3] = 0u;
    philox4x32_10(w, (uint32_t)(seed & 0xffffffffull), (uint32_t)(seed >> 32));
}

// Two draws of one (agent, step) side by side.  Unrolled, they share the first round's products and leave out
// the words of the second that the caller drops, and the step kernel's 80 registers hold them: 1M-agent metro
// 24.4 -> 23.5 ms, 32x32 lattice 16.3 -> 15.8, against a rolled loop.
__device__ __forceinline__ void draw4x2(uint64_t seed, int agent, int step, uint32_t ctr_a, uint32_t ctr_b, uint32_t a[4],
                                        uint32_t b[4])
{
    uint32_t k0 = (uint32_t)(seed & 0xffffffffull), k1 = (uint32_t)(seed >> 32);
    a[0] = b[0] = (uint32_t)agent; a[1] = b[1] = (uint32_t)step; a[2] = ctr_a; b[2] = ctr_b; a[3] = b[3] = 0u;
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t p0 = (uint64_t)0xD2511F53u * a[0], p1 = (uint64_t)0xCD9E8D57u * a[2];
        const uint64_t q0 = (uint64_t)0xD2511F53u * b[0], q1 = (uint64_t)0xCD9E8D57u * b[2];
        const uint32_t a1 = a[1], a3 = a[3], b1 = b[1], b3 = b[3];
        a[0] = (uint32_t)(p1 >> 32) ^ a1 ^ k0; a[1] = (uint32_t)p1; a[2] = (uint32_t)(p0 >> 32) ^ a3 ^ k1; a[3] = (uint32_t)p0;
        b[0] = (uint32_t)(q1 >> 32) ^ b1 ^ k0; b[1] = (uint32_t)q1; b[2] = (uint32_t)(q0 >> 32) ^ b3 ^ k1; b[3] = (uint32_t)q0;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
}

// Gumbel(0,1) from the top 24 bits: U = (k + 1/2) 2^-24 lies in (0,1).
__device__ __forceinline__ double gumbel_of(uint32_t w)
{
    const double U = ((double)(w >> 8) + 0.5) * (1.0 / 16777216.0);
    return -log(-log(U));
}

// The same draw in single precision, without branches.  With k = w >> 8,
// U = (k + 1/2) 2^-24.  For U < 1/2 the inner value y = -ln U is at least
// ln 2, and U is exact in float, so the hardware log2 (a few ulp) keeps y
// within ~3e-7 relative.  For U >= 1/2, e = 1 - U = (2^25 - 2k - 1) 2^-25 is
// an odd integer below 2^24 times a power of two, exact in float, and
// y = -ln(1 - e) takes Kahan's log1p correction (Goldberg, "What every
// computer scientist should know about floating-point arithmetic", 1991,
// Theorem 4): with u = fl(1 - e), whose distance 1 - u to one is exact,
// -ln(1 - e) = -ln(u) e / (1 - u) to a few ulp, and y = e when u rounds to
// one.  Both halves share one log of u.  The outer log then adds a few ulp of
// |g| <= 18, so |g - g_double| < 1e-5 (checked exhaustively over all 2^24
// values of k).  A decision compares two scores, each within that bound of
// its double value, and is taken on them only when it wins by kFastMargin
// (five times the largest possible error of the difference); otherwise it is
// recomputed with gumbel_of, so every decision equals the double-precision one.
__device__ __forceinline__ float gumbel_fast(uint32_t w)
{
    constexpr float kLn2 = 0.693147180559945f;
    const uint32_t k = w >> 8;
    const bool lower = k < (1u << 23);
    const float U = ((float)k + 0.5f) * (1.0f / 16777216.0f);
    const float e = (float)((1u << 25) - 2u * k - 1u) * (1.0f / 33554432.0f);   // 1 - U on the upper half
    const float u = lower ? U : 1.0f - e;
    const float lnu = __builtin_amdgcn_logf(u) * kLn2;
    const float r = lower ? 1.0f : e * __builtin_amdgcn_rcpf(1.0f - u);
    const float y = (!lower && u == 1.0f) ? e : -lnu * r;
    return -__builtin_amdgcn_logf(y) * kLn2;
}
constexpr double kFastMargin = 1e-4;

// The step, reverse and straight-through kernels read the state descriptor from device memory: it changes
// rarely, and as a kernel argument its 900 bytes would be written and fetched cold for every launch (an
// empty launch takes 2.6 us, one with 1 KB of arguments 4.0 us).  They are split into roles, each an
// inlined copy of code that reads the same fields; the optimiser would merge those loads into one at the
// kernel's entry and keep it live, in spilled scalar registers, through every role.  Each role therefore
// takes its own copy of the pointer, passed through an empty asm statement the optimiser cannot see
// through.  The constant address space keeps the loads scalar (nothing in these kernels writes it).
__device__ __forceinline__ const Dev &role_args(const Dev *dev)
{
    using ConstDev = const __attribute__((address_space(4))) Dev;
    ConstDev *p = (ConstDev *)dev;
    asm volatile("" : "+s"(p));
    return *(const Dev *)p;
}

// ---------------------------------------------------------------------------
// One step: car-following on every link and the node model at every node, side
// by side in one launch.
//
// Neither needs a result of the other.  The heads of a link have no leader
// (rank < lanes), so a node finds their arrival from their positions; what it
// needs from the links that leave it is their free entry slots, which it counts
// from the last `lanes` agents and their leaders.  So that nobody reads what
// somebody else writes, a step reads one copy of the positions and ring
// counters and writes another:
//   the link: the position of every agent on it;
//   its head node: head counter, bucket, outflow;
//   its tail node: tail counter, and the slots behind it (position 0, agent,
//     route row) of the agents that enter; a ring keeps `lanes` slots free, so
//     those are never slots that the link moves.
// A recording step reads tape entry k and writes entry k + 1, so the tape
// costs it no store of its own.
//
// Links (one lane group each)
//   Newell car-following with the link cap (Methods eq. newell_model; SI-A),
//   position form x' = min(x + u dt, max(x, x_lead - dn/kappa)), x_hat =
//   min(x', L); leader = rank - lanes, taken from the lane group's registers;
//   detector crossings, order check.
// Nodes (one lane group each, G >= candidates and out-links)
//   Arrival of the heads (x_hat >= L - 0.01); token accrual (the previous
//   step's idle cap min(B, 1) is applied here); vacancy of the out-links (entry
//   slots = lanes - #(x_hat <= dn/kappa)); releases into the origin queues.
//   Route choice of every candidate (heads of the in-links and origin fronts;
//   SI-B link choice: utility beta/c - theta*(t_ff + shortest time from the
//   link's head), hard choice argmax(V + Gumbel), ties to the lower candidate
//   index; a head whose link ends at its destination leaves the network);
//   merge per out-link (top-k by alpha_from + Gumbel, k = entry slots; SI-B
//   merge choice); FIFO resolve of each in-link's heads against its token
//   bucket; grafted transfer (SI-B eq. transfer; the graft itself lives in the
//   adjoint).
// Candidate lanes: the heads of in-link q take lanes [off_q, off_q + lanes_q),
// then the node's origins.
//
// Bound: a node wavefront's dependent chain of loads and instructions (13,000
// cycles alone on its SIMD, 17,000 on a full chip; a link wavefront takes 2,600
// to 5,500), not bytes (a 1M-agent step moves ~10 MB).  Hence links and nodes
// side by side, every load issued as soon as its address is known, no spilled
// registers (6 wavefronts a SIMD; with 7 the node's spills cost 20 %), and one
// copy of the code for every lane-group size.  Against a launch whose workgroups
// did their links first and their nodes after a barrier: 1M-agent metro 18.3 ->
// 13.5 us a step, 32x32 lattice 10.3 -> 9.0, 16 scenarios of 50k agents with
// their adjoint 79.6 -> 68.8 ms, 100-link network with its gradient 50.0 -> 41.2.
// ---------------------------------------------------------------------------
constexpr int kLinkUnroll = 4;   // rounds of a lane group whose positions are requested together
constexpr int kRevUnroll = 4;    // the same in the reverse: positions and adjoints

// A work item (link or node) is served by a lane group: G consecutive lanes of a wavefront (8, 16, 32 or
// 64, the same for every group of the wavefront).  All cross-lane traffic stays inside the group, and loops
// that contain shuffles have group-uniform trip counts.
struct Lanes {
    int G, gl, gbase;
    unsigned long long gm;
    __device__ __forceinline__ explicit Lanes(int G_) : G(G_)
    {
        const int l = lane_id();
        gl = l & (G - 1);
        gbase = l & ~(G - 1);
        gm = ~0ull >> (64 - G);
    }
    __device__ __forceinline__ unsigned long long mask(bool p) const { return (__ballot(p) >> gbase) & gm; }
    __device__ __forceinline__ int count(bool p) const { return __popcll(mask(p)); }
    template <class T>
    __device__ __forceinline__ T sum(T v) const
    {
        for (int o = G >> 1; o > 0; o >>= 1) v += __shfl_xor(v, o);
        return v;
    }
    // two sums over the group at once, in every lane: halves of 64 and 32 lanes by shuffles, the steps within 16 lanes
    // by DPP moves, which spare the shuffles' LDS latency (mirroring lanes whose quarters or halves already agree
    // exchanges them with the others)
    template <int kCtrl>
    static __device__ __forceinline__ double dpp(double v)
    {
        const long long b = __builtin_bit_cast(long long, v);
        const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)b, kCtrl, 0xf, 0xf, false);
        const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), kCtrl, 0xf, 0xf, false);
        return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
    }
    __device__ __forceinline__ void sum2(double &a, double &b) const
    {
        for (int o = G >> 1; o >= 16; o >>= 1) { const double p = __shfl_xor(a, o), q = __shfl_xor(b, o); a += p; b += q; }
        constexpr int kSwap1 = 0xb1, kSwap2 = 0x4e, kHalfMirror = 0x141, kMirror = 0x140;
        a += dpp<kSwap1>(a); b += dpp<kSwap1>(b);
        a += dpp<kSwap2>(a); b += dpp<kSwap2>(b);
        a += dpp<kHalfMirror>(a); b += dpp<kHalfMirror>(b);
        if (G >= 16) { a += dpp<kMirror>(a); b += dpp<kMirror>(b); }
    }
    template <class T>
    __device__ __forceinline__ T from(T v, int lane) const { return __shfl(v, gbase + lane); }
};

// Orders a wavefront's LDS accesses: they are carried out in program order, so the compiler alone has to
// keep it.  (A workgroup-scope fence would also wait for every global load and store in flight, 1-3 us
// after the stores of a step.)
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ float cf_update(float x, float xl, bool has_leader, float vf, float sp, float Lj)
{
    const float xf = x + vf;
    const float xc = xl - sp;
    const float cc = (x > xc) ? x : xc;
    const float xn = (has_leader && !(xf <= cc)) ? cc : xf;
    return (xn > Lj) ? Lj : xn;
}

// What a node's lanes publish to one another through LDS
struct alignas(8) CandRec { float kf; int ch; };   // candidate lane: its key and choice
struct alignas(8) OutRec {                         // out-link lane
    double util;
    int om, head, slots, tail;
    int place, base, cap, dep;                     // ring slot of the next entrant; departures of this step
    float u, pad;                                  // free speed (recording handles)
};

struct alignas(8) InRec {      // in-link lane: accrued level and its tangent, capacity multiplier, token rate m q lanes
    double B, dB, m, mqn;      // (the last three on recording handles),
    int64_t E;                 // outflow,
    int head, hm, cap, link;   // head counter and its slot, ring capacity, link
};

// what a node lane counts: releases of its origin, its candidate's outcome, a stuck head of its in-link
enum { NF_DEPARTED = 1, NF_EXITED = 2, NF_TRANSFERS = 4, NF_TIE_CHOICE = 8, NF_TIE_MERGE = 16 };
struct NodeCount { int released, flags, stuck; };

// where a step reads the state at its time and writes the state after it
struct StepAt {
    const float *pos_in;
    float *pos_out, *pos_copy;       // copy: tape entry of the state at t where it is not there already, or null
    const int4 *seg_in;
    int4 *seg_out, *seg_copy;
};

// element at a 32-bit byte offset from a pointer that is the same for the whole wavefront: one register and
// no 64-bit address arithmetic per access (a scenario's ring slots are below 2^30, so 4-byte elements fit)
template <class T>
__device__ __forceinline__ T &at32(T *p, uint32_t off)
{
    return *reinterpret_cast<T *>((char *)p + off);
}
template <class T>
__device__ __forceinline__ const T &at32(const T *p, uint32_t off)
{
    return *reinterpret_cast<const T *>((const char *)p + off);
}

// car-following of links [j0, j0 + count) of scenario s, one lane group of G lanes each
__device__ __forceinline__ void link_task(const Dev &d, const StepAt &io, int G, int s, int j0, int count, int sample_b)
{
    const Lanes g(G);
    const int gl = g.gl, gi = g.gbase >> __builtin_ctz(G);
    if (gi >= count) return;
    const int seg = s * d.L + j0 + gi;
    const LinkCf lc = d.lcf[seg];
    const int4 sg = io.seg_in[seg];
    const int cap = lc.cap, ln = lc.lanes;
    const int hm = sg.y, n_raw = sg.z - sg.x;
    const int n = min(n_raw, cap);   // an overflowing ring (flagged below) is never read past its end
    const int64_t sR = (int64_t)s * d.ring_total;
    const float *pos_in = io.pos_in + sR;
    float *pos_out = io.pos_out + sR, *pos_copy = io.pos_copy ? io.pos_copy + sR : nullptr;
    const float vf = lc.vf, sp = lc.sp, Lj = lc.L;
    // byte offset of rank r's slot
    const uint32_t first_off = (uint32_t)(lc.ring_base + hm) * 4u;
    auto off_of = [&](int r) { return first_off + 4u * (uint32_t)(hm + r >= cap ? r - cap : r); };
    if (io.seg_copy && gl == 0) io.seg_copy[seg] = sg;
    // a ring keeps `lanes` slots free, so an entry slot never aliases a slot live one step earlier
    if (gl == 0 && n_raw > cap - ln) atomicOr(&d.err[ERR_RING_OVERFLOW], 1);
    constexpr int U = kLinkUnroll, P = 2;   // rounds of loads in flight; rounds worked on together
    int viol = 0;
    float xprev = 0.f;
    const int lsrc = g.gbase + ((gl - ln) & (G - 1)), psrc = g.gbase + ((gl - 1) & (G - 1));
    const bool lsend = gl >= G - ln, psend = gl == G - 1;
    for (int r0 = 0; r0 < n; r0 += U * G) {
        float xu[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int r = r0 + q * G + gl;
            xu[q] = r < n ? at32(pos_in, off_of(r)) : 0.f;
        }
#pragma unroll
        for (int p = 0; p < U; p += P) {
            if (r0 + p * G >= n) break;
            float xl[P], xp[P];
            // rank r - lanes and rank r - 1: from this round's lanes, or the previous round's last ones
#pragma unroll
            for (int q = 0; q < P; ++q) {
                const float x = xu[p + q], y = p + q ? xu[p + q ? p + q - 1 : 0] : xprev;
                xl[q] = __shfl(lsend ? y : x, lsrc);
                xp[q] = __shfl(psend ? y : x, psrc);
            }
#pragma unroll
            for (int q = 0; q < P; ++q) {
                const int r = r0 + (p + q) * G + gl;
                const float x = xu[p + q], xh = cf_update(x, xl[q], r >= ln, vf, sp, Lj);
                if (r < n) {
                    at32(pos_out, off_of(r)) = xh;
                    if (pos_copy) at32(pos_copy, off_of(r)) = x;
                    // the step's input order (entrants of the previous step included): position descending
                    viol += (r > 0) & (xp[q] < x);
                }
            }
        }
        xprev = xu[U - 1];
    }
    if (g.count(viol > 0)) {
        viol = g.sum(viol);
        if (gl == 0)
            atomicAdd((unsigned long long *)&d.ctr[((int64_t)s * kCtrSlots) * CTR_N + CTR_ORDER_VIOL],
                      (unsigned long long)viol);
    }
    // detector crossings, on sampling steps only: the updated positions once more.  The head counter is the
    // outflow so far (both start at 0 and count the agents that left).
    const int nd = sample_b >= 0 ? (lc.det >> 24) : 0;
    for (int k = 0; k < nd; ++k) {
        const int det = d.det_list[(lc.det & 0xffffff) + k];
        const float at = d.det_pos[det];
        int cnt = 0;
        for (int r = gl; r < n; r += G) {
            const float x = at32(pos_in, off_of(r)), xl = r >= ln ? at32(pos_in, off_of(r - ln)) : 0.f;
            cnt += cf_update(x, xl, r >= ln, vf, sp, Lj) >= at;
        }
        cnt = g.sum(cnt);
        if (gl == 0) d.cum[((int64_t)s * d.D + det) * d.nb + sample_b] = sg.x + cnt;
    }
}

// Whole-ring counts of links [j0, j0 + count) for rings out of position order: after the update of step t, the
// agents on the entry slots and the agents that arrive.
__device__ __forceinline__ void count_task(const Dev &d, const float *pos_in, const int4 *seg_in, int G, int s, int j0, int count)
{
    const Lanes g(G);
    const int gl = g.gl, gi = g.gbase >> __builtin_ctz(G);
    if (gi >= count) return;
    const int seg = s * d.L + j0 + gi;
    const LinkCf lc = d.lcf[seg];
    const int4 sg = seg_in[seg];
    const int cap = lc.cap, ln = lc.lanes, hm = sg.y, n = min(sg.z - sg.x, cap);
    const float *pos = pos_in + (int64_t)s * d.ring_total;
    const uint32_t first_off = (uint32_t)(lc.ring_base + hm) * 4u;
    auto at = [&](int r) { return at32(pos, first_off + 4u * (uint32_t)(hm + r >= cap ? r - cap : r)); };
    int taken = 0, arrived = 0;
#pragma unroll 4
    for (int r = gl; r < n; r += G) {
        const float xh = cf_update(at(r), r >= ln ? at(r - ln) : 0.f, r >= ln, lc.vf, lc.sp, lc.L);
        taken += xh <= lc.sp;
        arrived += xh >= lc.thr;
    }
    taken = g.sum(taken);
    arrived = g.sum(arrived);
    if (gl == 0) d.ring_cnt[seg] = make_int2(taken, arrived);
}

// What a step kernel does about rings out of position order (Dev::disorder): knows that there are none; reads the
// whole-ring counts of count_task, if the descriptor says so; has its nodes look at whole rings, if it says so.  The
// one-workgroup kernel without the checks saves 1 to 2 % of a step where the host knows the order; a step that is a
// launch of its own gains nothing by it (metro 0.5 % slower, 32x32 lattice 1.5 % faster).
enum { kOrdered, kCounted, kScan };

// The node model at node v.  `orc`, `crc` and `ckey` are the lane group's own entries.
template <int kRings>
__device__ __forceinline__ NodeCount node_work(const Dev &d, const StepAt &io, const Tape &tp, const Lanes &g, int s,
                                               int v, int t, int tape_k, InRec *inr, OutRec *orc, CandRec *crc, double *ckey)
{
    const int gl = g.gl, G = g.G;
    const int64_t sL = (int64_t)s * d.L, sR = (int64_t)s * d.ring_total;
    // ---- loads, level by level, each issued together (padded tables need no offsets; a lane without a role
    // reads a valid stand-in entry and its result is selected away) ----
    const int cnt = d.node_cnt[v];
    const int om = max(d.out_pad[(int64_t)v * d.max_out + min(gl, d.max_out - 1)], 0);
    // (in-link, q | rank << 8) on head lanes, (origin, first queue entry) on origin lanes
    const int2 cm = d.cand[(int64_t)v * d.max_cand + min(gl, d.max_cand - 1)];
    const int jin = max(d.in_pad[(int64_t)v * d.max_in + min(gl, d.max_in - 1)], 0);
    // first head lane of in-link gl
    const int off_res = d.in_loff[(int64_t)v * d.max_in + min(gl, d.max_in - 1)] & (kWave - 1);
    const int64_t rbase = d.route_base[v];
    const int ndidx = d.node_didx[v];
    const bool ste_rec = tape_k >= 0 && tp.ste != nullptr;      // straight-through tape
    const int cb = ste_rec ? d.cbase[v] : 0;
    const uint64_t seed = d.seed[s];
    const int deg = cnt & 0xff, dego = (cnt >> 8) & 0xff, ncin = (cnt >> 24) & 0xff, nc = ncin + ((cnt >> 16) & 0xff);
    const bool head_lane = gl < ncin, org_lane = gl >= ncin && gl < nc;
    const int qi = cm.y & 0xff, hr_r = cm.y >> 8;   // head lanes: in-link index, rank
    const int from = head_lane ? cm.x : -1;
    const int64_t cj = sL + (head_lane ? cm.x : 0);
    // second level
    const LinkCf hc = d.lcf[cj];
    const int4 hs = io.seg_in[cj];
    const LinkNd &fc = d.lnd[cj];
    const float falpha = fc.alpha;
    const int ftl = fc.tail;
    const LinkCf lc = d.lcf[sL + om];
    const LinkNd &oc = d.lnd[sL + om];
    const double util = oc.util;
    const int ohead = oc.head;
    const int4 sg = io.seg_in[sL + om];
    const float ou = d.dB ? d.u[sL + om] : 0.f;
    const LinkSt li = d.ls[sL + jin];
    const int4 si = io.seg_in[sL + jin];
    const double acc = d.acc[sL + jin];
    {   // token accrual of the in-links (after the previous step's idle cap).  What a lane needs again only at the
        // end waits in LDS: registers held across the whole node would cost occupancy.
        InRec r{(li.B > 1.0 ? 1.0 : li.B) + acc, 0.0, 0.0, 0.0, li.E, si.x, si.y, d.cap[jin], jin};
        if (d.dB) {   // tangent of the level in the multiplier; the idle cap clears it
            const double q = (double)d.capacity[jin], ln = (double)d.lanes[jin];
            r.m = (double)d.capm[sL + jin];
            r.dB = (li.B > 1.0 ? 0.0 : d.dB[sL + jin]) + q * ln * d.dt;
            if (gl < deg) d.dB[sL + jin] = r.dB;
            r.mqn = r.m * q * ln;
        }
        inr[gl] = r;
    }
    const int qb = cm.y, so = s * d.O + (org_lane ? cm.x : 0);
    int rel = 0, dp0 = 0, qn = 0;
    double D = 0.0, incr = 0.0;
    const double t1 = (t + 1) * d.dt;
    if (org_lane) {   // release and departure pointers, queue length, this step's departures
        rel = d.rel_ptr[so];
        dp0 = d.dep_ptr[so];
        qn = d.q_off[cm.x + 1] - qb;
        if (!d.fixed_mode) {
            D = d.Dacc[so];
            // bins are whole numbers of steps: step t lies in bin t / steps_per_bin, and only its
            // neighbours can touch the step through rounding of the bin edges (bins in increasing
            // order, as a sum over all bins would add them)
            const double t0 = t * d.dt;
            const int bc = t / d.rate_bin_steps;
            for (int b = max(bc - 1, 0); b <= bc + 1 && b < d.n_rate_bins; ++b) {
                const double lo = fmax(b * d.rate_bin_s, t0), hi = fmin((b + 1) * d.rate_bin_s, t1);
                if (hi > lo) incr += (double)d.rates[(int64_t)so * d.n_rate_bins + b] * (hi - lo);
            }
        }
    }
    // third level: the heads, which have no leader (rank < lanes), so the node finds their arrival itself;
    // the queue's front, whether or not this step releases it
    const int hcap = hc.cap, hn = min(hs.z - hs.x, hcap);
    const bool in_ring = head_lane && hr_r < hn;
    const int hp = hs.y + hr_r, hslot = hp >= hcap ? hp - hcap : hp;   // ring slot of this head
    const uint32_t hoff = in_ring ? (uint32_t)(hc.ring_base + hslot) * 4u : 0u;
    int ag = -1, didx = 0;
    float hx = 0.f;
    if (in_ring) {
        hx = at32(io.pos_in + sR, hoff);
        ag = at32(d.ring_agent + sR, hoff);
        didx = at32(d.ring_aux + sR, hoff);
    } else if (org_lane && dp0 < qn) {
        ag = d.q_list[qb + dp0];
        didx = d.q_didx[qb + dp0];
    }
    if (gl < dego) {   // entry slots of the out-link
        const int cap = lc.cap, ln = lc.lanes, hm = sg.y, n = min(sg.z - sg.x, cap);
        const float *pos = io.pos_in + sR;
        const uint32_t first_off = (uint32_t)(lc.ring_base + hm) * 4u;
        auto at = [&](int r) { return at32(pos, first_off + 4u * (uint32_t)(hm + r >= cap ? r - cap : r)); };
        int occ = 0;
        // an ordered ring: at most `lanes` agents matter, and they are the last ones
        const int span = kRings == kScan && d.disorder ? n : min(n, ln);
        for (int i0 = 0; i0 < span; i0 += 4) {
            float x[4], xl[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = n - 1 - (i0 + q);
                const bool in = i0 + q < span;
                x[q] = in ? at(r) : 0.f;
                xl[q] = in && r >= ln ? at(r - ln) : 0.f;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                occ += (i0 + q < span) & (cf_update(x[q], xl[q], n - 1 - (i0 + q) >= ln, lc.vf, lc.sp, lc.L) <= lc.sp);
        }
        if (kRings == kCounted && d.disorder) occ = d.ring_cnt[sL + om].x;
        const int place = hm + n;
        orc[gl] = OutRec{util, om, ohead, max(0, ln - occ), sg.z, place >= cap ? place - cap : place, lc.ring_base, cap, 0, ou, 0.f};
    }
    // heads of each in-link: its arrivals come first in an ordered ring
    int h;
    {
        const int hl = hc.lanes;
        const bool arr = in_ring && cf_update(hx, 0.f, false, hc.vf, hc.sp, hc.L) >= hc.thr;
        const unsigned long long first = g.mask(arr) >> ((gl - hr_r) & (kWave - 1));
        h = __popcll(first & ((1ull << hl) - 1ull));
        if (kRings == kCounted && d.disorder) h = min(d.ring_cnt[cj].y, hl);
        if (kRings == kScan && d.disorder) {   // a caller's placement may have left one out of order: all of the ring's arrivals
            int a = 0;
            for (int r = hr_r; head_lane && r < hn; r += hl) {   // this lane's ranks lead one another
                auto at = [&](int k) {
                    const int p = hs.y + k;
                    return at32(io.pos_in + sR, (uint32_t)(hc.ring_base + (p >= hcap ? p - hcap : p)) * 4u);
                };
                a += cf_update(at(r), r >= hl ? at(r - hl) : 0.f, r >= hl, hc.vf, hc.sp, hc.L) >= hc.thr;
            }
            h = 0;
            for (int k = 0; k < kMaxLanes; ++k) {
                const int b = g.from(a, (gl - hr_r + k) & (G - 1));
                h += k < hl ? b : 0;
            }
            h = min(h, hl);
        }
        if (head_lane && hr_r >= h) ag = -1;
    }
    // ---- releases of this step ----
    int released = 0;
    if (org_lane) {
        int newrel = rel;
        double rr = 1.0;
        if (d.fixed_mode) {
            while (newrel < qn && d.q_rstep[qb + newrel] <= (int64_t)t) ++newrel;
        } else {
            D += incr;
            if (incr != 0.0) d.Dacc[so] = D;
            rr = incr / d.dt;
            while (newrel < qn && (double)(newrel + 1) <= D) ++newrel;
        }
        // mark the released agents, four queue entries loaded per round before their writes
        for (int k0 = rel; k0 < newrel; k0 += 4) {
            int a4[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) a4[q] = (k0 + q < newrel) ? d.q_list[qb + k0 + q] : -1;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (a4[q] < 0) continue;
                const int64_t ga = (int64_t)s * d.N + a4[q];
                d.status[ga] = AG_QUEUED;
                if (!d.fixed_mode) d.tstar[ga] = t1 - (D - (double)(k0 + q + 1)) / rr;
                d.rel_t[ga] = t;
            }
        }
        if (newrel != rel) d.rel_ptr[so] = newrel;
        released = newrel - rel;
        if (dp0 >= newrel) ag = -1;
    }
    wave_lds_sync();
    uint32_t small = 0;   // NF_* flags
    const int64_t ste_i = ((int64_t)tape_k * d.S + s) * d.n_cand + cb + gl;
    int np = 0, nent = 0, n_stuck = 0;
    double Bj = inr[gl].B;
    if (g.count(ag >= 0) == 0) {   // nothing to move at this node this step
        if (ste_rec && gl < nc) tp.ste[ste_i] = make_int4(-1, 0, -1, -1);
    } else {

    // ---- route choice (group-uniform loop over chunks of out-links) ----
    const bool exiting = ag >= 0 && head_lane && didx == ndidx;
    const bool chooser = ag >= 0 && !exiting;
    const double *route = d.route + rbase + (int64_t)didx * dego;   // this head's row
    const int ftail = head_lane ? ftl : -1;
    // fast pass on single-precision noise: for each chunk of out-links, every route entry and
    // Philox word of the chunk is requested before the first score, so one memory round trip
    // serves the chunk
    double best = -INFINITY, second = -INFINITY;
    int arg = CH_STUCK, argk = 0;   // chosen link and its index among the node's out-links
    uint32_t wm = 0u;               // merge-key word: independent of the choice
    for (int c0 = 0; c0 == 0 || c0 < dego; c0 += 4) {
        double rt[4];
        uint32_t w[4], w2[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) rt[q] = (chooser && c0 + q < dego) ? route[c0 + q] : INFINITY;
        // choice block c0 / 4 (purpose 0) and, the first time, the merge draw (purpose 1)
        if (ag >= 0) draw4x2(seed, ag, t, 2u * (uint32_t)(c0 >> 2), 1u, w, w2);
        if (c0 == 0) wm = w2[0];
        if (!chooser) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (c0 + q >= dego) break;
            const OutRec &o = orc[c0 + q];
            const bool ok = !((!d.allow_uturn) & head_lane & (o.head == ftail)) & (rt[q] < INFINITY);
            const double sc = o.util - d.theta * rt[q] + (double)gumbel_fast(w[q]);
            const bool top = ok & (sc > best), sec = ok & !top & (sc > second);
            second = top ? best : (sec ? sc : second);
            best = top ? sc : best;
            arg = top ? o.om : arg;
            argk = top ? c0 + q : argk;
        }
    }
    // lanes whose winner is not clear on the fast noise redo the choice in double precision (rare)
    const bool redo = chooser && second > -INFINITY && best - second < kFastMargin;
    if (redo) {
        best = -INFINITY;
        second = -INFINITY;
        arg = CH_STUCK;
        argk = 0;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll 1
        for (int c = 0; c < dego; ++c) {
            if ((c & 3) == 0) { uint32_t u[4]; draw4x2(seed, ag, t, 2u * (uint32_t)(c >> 2), 1u, w, u); }
            const uint32_t wc = w[0];
            w[0] = w[1]; w[1] = w[2]; w[2] = w[3];
            const OutRec &o = orc[c];
            const double rt = route[c];
            if (!d.allow_uturn && head_lane && o.head == ftail) continue;
            if (!(rt < INFINITY)) continue;
            const double V = o.util - d.theta * rt;
            const double sc = V + gumbel_of(wc);
            if (sc > best) { second = best; best = sc; arg = o.om; argk = c; }
            else if (sc > second) second = sc;
        }
    }
    int ch = CH_NONE;
    if (chooser) {
        ch = arg;
        if (arg >= 0 && second > -INFINITY && best - second < 1e-12 * (1.0 + fabs(best))) {
            small |= NF_TIE_CHOICE;
            tie_record(d, s, t, TIE_CHOICE, ag, arg, arg);
        }
    } else if (exiting) {
        ch = CH_EXIT;
    }
    // ---- merge: rank among candidates wanting the same link ----
    // Every candidate lane publishes (key, choice, agent); a chooser counts the candidates of its own
    // out-link that precede it in key order.  Fast pass on single-precision keys alpha_from + g' (g'
    // the fast noise): each lies within 1e-5 + 2^-24 |key| of the double-precision key, so while
    // |key| < 512 a difference of two keys is off by less than 8.2e-5 and its sign is exact wherever
    // it exceeds kFastMargin.  A group with a rival pair inside the margin, or a key of 512 or more,
    // ranks again on double-precision keys (ties broken by agent id, and the near-tie log, live only
    // there).  The candidate lanes 0..nc-1 go in chunks of four, each chunk unrolled and
    // branch-free (predicates combine with non-short-circuit & and |, so no record read is placed
    // under a branch) so that its broadcast LDS reads are in flight together; lanes past nc are
    // masked out of the sums.
    // The bits of `ahead` (candidates of the same link ranked before this one) and `wants` (candidates
    // whose choice is out-link gl) serve the merge now and, restricted to those that pass, the entry
    // order and the entrants later.
    const double alpha = head_lane ? (double)falpha : 1.0;
    const float kf = ag >= 0 ? (float)alpha + gumbel_fast(wm) : 0.f;
    const bool act = ag >= 0 && ch >= 0;
    const int me_k = act ? argk : -1;
    unsigned long long ahead = 0, wants = 0;
    bool close = false;
    crc[gl] = CandRec{kf, me_k};
    wave_lds_sync();
    int kn = act & !(fabsf(kf) < 512.f);
    for (unsigned long long left = g.mask(act); left;) {   // four choosers a round, their records read together
        int e[4];
        CandRec o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            e[k] = left ? __builtin_ctzll(left) : -1;
            left &= left - 1;
            o[k] = crc[max(e[k], 0)];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const bool rival = act & (e[k] >= 0) & (e[k] != gl) & (o[k].ch == me_k);
            const float diff = o[k].kf - kf;
            const unsigned long long bit = 1ull << (e[k] & 63);
            ahead |= (rival & (diff > 0.f)) ? bit : 0ull;
            wants |= ((e[k] >= 0) & (o[k].ch == gl)) ? bit : 0ull;
            kn |= rival & (fabsf(diff) < (float)kFastMargin);
        }
    }
    if (g.count(kn != 0) != 0) {   // the group's ranks on double-precision keys
        const double key = ag >= 0 ? alpha + gumbel_of(wm) : 0.0;
        ckey[gl] = key;
        wave_lds_sync();
        const double tol = 1e-12 * (1.0 + fabs(key));
        ahead = 0;
        for (int e = 0; e < nc; ++e) {
            const double diff = ckey[e] - key;   // exact in sign: a key is ahead iff diff > 0
            const bool rival = act & (e != gl) & (crc[e].ch == me_k);
            const bool first = (diff > 0.0) | ((diff == 0.0) & (g.from(ag, e) < ag));
            ahead |= (unsigned long long)(rival & first) << e;
            close |= rival & !first & (-diff < tol);
        }
    }
    const int sl = act ? orc[argk].slots : 0;
    const bool won = act && __popcll(ahead) < sl;
    if (close) {
        small |= NF_TIE_MERGE;
        tie_record(d, s, t, TIE_MERGE, ag, ch, 1);
    }

    // ---- resolve: lane q < deg walks in-link q's heads in rank order; their outcomes as bits ----
    const unsigned long long m_exit = g.mask(ch == CH_EXIT), m_won = g.mask(won), m_stuck = g.mask(ch == CH_STUCK);
    {
        const uint32_t x = (uint32_t)(m_exit >> off_res), y = (uint32_t)(m_won >> off_res);
        int nh = g.from(h, off_res & (G - 1));   // <= lanes <= kMaxLanes
        nh = gl < deg ? nh : 0;
        bool stop = false;
        for (int r = 0; r < nh && !stop; ++r) {
            if ((x >> r) & 1u) ++np;
            else if (((y >> r) & 1u) && Bj >= 1.0) { Bj -= 1.0; ++np; }
            else { stop = true; n_stuck = (int)(m_stuck >> (off_res + r)) & 1; }
        }
    }
    const int np_q = g.from(np, qi & (G - 1));
    const bool passed = head_lane ? (ag >= 0) && hr_r < np_q : won;

    // ---- entrants per out-link (lane k < dego counts link k's) and each entrant's place in key order ----
    // (entrants onto one link are rivals of one another)
    const bool entering = passed && act;
    const unsigned long long m_in = g.mask(entering);
    nent = __popcll(wants & m_in);
    const int erank = __popcll(ahead & m_in);
    int slot = 0;   // ring slot (of this scenario) the entrant takes
    if (entering) {
        const OutRec &o = orc[argk];
        const int p = o.place + erank;
        slot = o.base + (p >= o.cap ? p - o.cap : p);
    }
    const int64_t ga = (int64_t)s * d.N + (ag >= 0 ? ag : 0);
    // admission graft: a head leaving on a token carries the token's availability
    // time t_tok = (t+1)dt - (B_pre - 1)/(m q n) into its entry position
    // (psi = -u_to t_tok); B_pre = accrued level minus the tokens taken ahead of it
    float gfac = 0.f;
    const bool graft = tape_k >= 0 && tp.dstg != nullptr;   // admission-graft tape
    if (graft) {
        // heads ahead on the link that chose an out-link (their lanes end right before this one)
        const int tok = __popcll((g.mask(act) >> (gl - hr_r)) & ((1ull << hr_r) - 1ull));
        if (passed && from >= 0 && ch >= 0) {
            const InRec &q = inr[qi];
            if (q.mqn > 0.0) {
                const double dtdm = -q.dB / q.mqn + (q.B - (double)tok - 1.0) / (q.m * q.mqn);
                gfac = (float)(-(double)orc[argk].u * dtdm);
            }
        }
    }
    if (ste_rec && gl < nc) {   // this candidate's choice, outcome and the ring slot its adjoint will hold at t+1
        int4 rec = make_int4(-1, 0, -1, -1);
        if (ag >= 0 && ch >= 0) {
            int loc = -1;
            if (passed) loc = slot;
            else if (from >= 0) loc = (int)(hoff >> 2);
            rec = make_int4(ag, argk | (min(sl, 255) << 8) | (passed << 16), from, loc);
        }
        tp.ste[ste_i] = rec;
    }
    if (tape_k >= 0 && passed && from >= 0) {   // where each leaving head went (-1: left the network)
        const int64_t ti = ((int64_t)tape_k * d.S * d.L + sL + from) * d.maxl + hr_r;
        tp.dst[ti] = ch >= 0 ? (int32_t)(sR + slot) : -1;
        if (graft) tp.dstg[ti] = gfac;
    }
    if (passed) {
        if (ch >= 0) {
            d.ring_agent[sR + slot] = ag;
            d.ring_aux[sR + slot] = didx;
            io.pos_out[sR + slot] = 0.f;
            if (!head_lane) {
                d.status[ga] = AG_ON;
                d.dep_t[ga] = t;
                // a departure: its entry order on the link and its agent, for the reverse's departure
                // grafts (erank < entry slots <= lanes <= kMaxLanes)
                if (tape_k >= 0) {
                    atomicOr(&orc[argk].dep, 1 << erank);
                    tp.agent[(int64_t)(tape_k + 1) * d.S * d.ring_total + sR + slot] = ag;
                }
                d.dep_ptr[so] = dp0 + 1;
                small |= NF_DEPARTED;
            } else {
                small |= NF_TRANSFERS;
            }
        } else {
            d.status[ga] = AG_EXITED;
            d.exit_t[ga] = t;
            small |= NF_EXITED;
        }
    }
    wave_lds_sync();
    }
    // ring counters after the step: the head of every in-link, the tail of every out-link
    if (gl < deg) {
        const InRec &r = inr[gl];
        const int64_t j = sL + r.link;
        const int p = r.hm + np;
        d.ls[j] = LinkSt{Bj, r.E + np};   // the idle cap min(B, 1) is applied at the next accrual
        *reinterpret_cast<int2 *>(&io.seg_out[j].x) = make_int2(r.head + np, p >= r.cap ? p - r.cap : p);
    }
    if (gl < dego) {
        const OutRec &o = orc[gl];
        *reinterpret_cast<int2 *>(&io.seg_out[sL + o.om].z) = make_int2(o.tail + nent, o.dep);
    }
    return NodeCount{released, (int)small, n_stuck};
}

// Counters of a wavefront's nodes: flags counted by ballot, then one atomic per non-zero counter into one
// of kCtrSlots slots (spread by item) so that concurrent wavefronts rarely hit the same address.
__device__ __forceinline__ void add_counters(const Dev &d, int s, int item, const NodeCount &c)
{
    unsigned long long *ctr = (unsigned long long *)&d.ctr[((int64_t)s * kCtrSlots + (item % kCtrSlots)) * CTR_N];
    const bool lead = lane_id() == 0;
    auto add = [&](int k, bool flag) {
        const unsigned long long b = __ballot(flag);
        if (b && lead) atomicAdd(ctr + k, (unsigned long long)__popcll(b));
    };
    add(CTR_DEPARTED, c.flags & NF_DEPARTED);
    add(CTR_EXITED, c.flags & NF_EXITED);
    add(CTR_TRANSFERS, c.flags & NF_TRANSFERS);
    add(CTR_STUCK, c.stuck);
    if (__ballot((c.flags & (NF_TIE_CHOICE | NF_TIE_MERGE)) != 0)) {   // rare
        add(CTR_TIES, c.flags & NF_TIE_CHOICE);
        add(CTR_TIES, c.flags & NF_TIE_MERGE);
    }
    if (__ballot(c.released != 0)) {
        int r = c.released;
        for (int o = 32; o > 0; o >>= 1) r += __shfl_xor(r, o);
        if (lead) atomicAdd(ctr + CTR_RELEASED, (unsigned long long)r);
    }
}

// Kernel timing (only when a launch has a record): every wave stores its start and end, read from the
// real-time counter, into its own pair of the launch's record (plain stores, no contention);
// k_stamp_reduce later folds a record into the first start and the last end, the kernel's
// execution interval without the dispatch gaps around it.
__device__ __forceinline__ unsigned long long stamp_begin(const unsigned long long *rec)
{
    return rec ? wall_clock64() : 0ull;
}
__device__ __forceinline__ void stamp_end(unsigned long long *rec, unsigned long long t0, int64_t w)
{
    if (!rec) return;
    const unsigned long long t1 = wall_clock64();
    if ((threadIdx.x & 63) == 0) {
        rec[2 * w] = t0;
        rec[2 * w + 1] = t1;
    }
}

// A launch's tasks per scenario: node tasks (a wavefront's nodes, 64 / lanes of one class, widest class first)
// and link tasks (64 / lanes links of one ring class, longest rings first).  Several workgroups: node task b is
// the first wavefront's of workgroup b, the others take the link tasks (two of them: an average node has about
// that many tasks of in-links.  With one, 16 scenarios of 50k agents slow down by 8 %, with three by 6 % and
// metro by 3 %; leaving out the idle first wavefronts of workgroups past the last node task gains nothing).
// kXcd = 3: each class's tasks go to the 8 XCDs in contiguous eighths, in whole rows of 8 workgroups.  kXcd = 0: a
// scenario's tasks in order, without rows, where these would be mostly idle (packed_roles).
// As kernel arguments: no chain of descriptor reads before a wavefront knows its work.
struct StepRoles {
    struct Role { int slot, first, n; } node[4], link[4];   // first slot of the role; first id, number of ids
    int blocks;                                             // workgroups per scenario
};

// nodes of a task
template <int kRings>
__device__ __forceinline__ void node_task(const Dev &d, const StepAt &at, const Tape &tp, int G, int s, int v0, int nv, int t,
                                          int tape_k, InRec *inr, OutRec *orc, CandRec *crc, double *ckey)
{
    const Lanes g(G);
    const int vi = g.gbase >> __builtin_ctz(G), o = g.gbase;
    NodeCount nc{0, 0, 0};
    if (vi < nv) nc = node_work<kRings>(d, at, tp, g, s, v0 + vi, t, tape_k, inr + o, orc + o, crc + o, ckey + o);
    add_counters(d, s, v0, nc);
}

// detector bin sampled by step t, or -1
__device__ __forceinline__ int sample_bin(const Dev &d, int t)
{
    return d.cbs > 0 && (t + 1) % d.cbs == 0 && (t + 1) / d.cbs <= d.nb ? (t + 1) / d.cbs - 1 : -1;
}

// the link task of slot q of a launch, if there is one: f(lanes a link, first link, links)
template <int kXcd, class F>
__device__ __forceinline__ void with_link_task(const StepRoles &roles, int q, int g_link, F &&f)
{
    constexpr int LW = kStepWaves - 1;
    int c = 0;
    StepRoles::Role R = roles.link[0];
#pragma unroll
    for (int k = 1; k < 4; ++k) {
        const StepRoles::Role &r = roles.link[k];
        const bool in = q >= r.slot;
        R = {in ? r.slot : R.slot, in ? r.first : R.first, in ? r.n : R.n};
        c = in ? k : c;
    }
    const int lanes = ring_lanes(3 - c, g_link), lp = 6 - __builtin_ctz(lanes);
    const int tasks = (R.n + (1 << lp) - 1) >> lp, per = (tasks + (1 << kXcd) - 1) >> kXcd;
    // slot i of the role: workgroup g of it, on XCD x
    const int i = q - R.slot, g = i / LW, x = g & ((1 << kXcd) - 1), k = (g >> kXcd) * LW + i % LW;
    const int j = (x * per + k) << lp;
    if (k < per && j < R.n) f(lanes, R.first + j, min(1 << lp, R.n - j));
}

// A launch before each step where a placement has left rings out of position order (Dev::disorder); the one-
// workgroup kernel counts between two barriers.  A node that looked at its whole rings itself, a few lanes a ring,
// took 124 us a step at a 64-candidate hub of rings of 100 agents (now 17), 59 at the 1M-agent metro with 400,000
// placed (33), 28.5 with rings of 96 on a 4 x 4 lattice (12.4).  Captured steps, which cannot know what a replay
// finds, have that way where a step is a launch (kScan).
template <int kXcd>
__global__ __launch_bounds__(kStepWaves * kWave)
void k_ring_counts(const Dev *dev, const float *pos_in, const int4 *seg_in, StepRoles roles, int g_link)
{
    int b = (int)blockIdx.x, s = 0;
    if (kXcd == 0 || (int)gridDim.x != roles.blocks) {
        const int S = (int)gridDim.x / roles.blocks;
        b /= S;
        s = (int)blockIdx.x - b * S;
    }
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (w > 0)
        with_link_task<kXcd>(roles, b * (kStepWaves - 1) + w - 1, g_link, [&](int lanes, int j, int n) {
            count_task(role_args(dev), pos_in, seg_in, lanes, s, j, n);
        });
}

template <int kRings, int kXcd>
__global__ __launch_bounds__(kStepWaves * kWave) __attribute__((amdgpu_waves_per_eu(6)))
void k_step(const Dev *dev, StepIo io, StepRoles roles, int g_link, int t, int tape_k)
{
    __shared__ InRec inr[kWave];
    __shared__ OutRec orc[kWave];
    __shared__ CandRec crc[kWave];
    __shared__ double ckey[kWave];   // double-precision merge keys (groups that rank exactly)
    // scenario-fastest: the workgroups with nodes, the longest, of every scenario come first (16 scenarios of 50k
    // agents, 1.7 times what the chip holds at once, with their adjoint 68.7 -> 61.7 ms)
    int b = (int)blockIdx.x, s = 0;
    if (kXcd == 0 || (int)gridDim.x != roles.blocks) {
        const int S = (int)gridDim.x / roles.blocks;
        b /= S;
        s = (int)blockIdx.x - b * S;
    }
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const StepAt at{io.pos_in, io.pos_out, io.pos_copy, io.seg_in, io.seg_out, io.seg_copy};
    // rows: the roles' first slots are multiples of 8, so b % 8 is the XCD, or for several scenarios decides on it
    if (w == 0) {
        const unsigned long long ts = stamp_begin(io.kstamp_node);
        int c = 0;
        StepRoles::Role R = roles.node[0];
#pragma unroll
        for (int k = 1; k < 4; ++k)
            if (b >= roles.node[k].slot) { R = roles.node[k]; c = k; }
        const int i = b - R.slot, tasks = (R.n + (1 << c) - 1) >> c, per = (tasks + (1 << kXcd) - 1) >> kXcd;
        const int k = ((i & ((1 << kXcd) - 1)) * per + (i >> kXcd)) << c;
        if ((i >> kXcd) < per && k < R.n)
            node_task<kRings>(role_args(dev), at, io.tape, kWave >> c, s, R.first + k, min(1 << c, R.n - k), t, tape_k, inr, orc, crc, ckey);
        stamp_end(io.kstamp_node, ts, blockIdx.x);
    } else {
        constexpr int LW = kStepWaves - 1;
        const unsigned long long ts = stamp_begin(io.kstamp);
        with_link_task<kXcd>(roles, b * LW + w - 1, g_link, [&](int lanes, int j, int n) {
            const Dev &d = role_args(dev);
            link_task(d, at, lanes, s, j, n, sample_bin(d, t));
        });
        stamp_end(io.kstamp, ts, blockIdx.x * LW + w - 1);
    }
}

// A small network (Dev::solo): one workgroup a scenario runs many steps, a barrier apart.
template <int kRings>
__global__ __launch_bounds__(kSoloWaves * kWave)
void k_step_solo(const Dev *dev, StepIo io, HomeIo home, int t0, int n_steps, int tape_k)
{
    constexpr int NL = kSoloNodeWaves * kWave;
    __shared__ InRec inr[NL];
    __shared__ OutRec orc[NL];
    __shared__ CandRec crc[NL];
    __shared__ double ckey[NL];
    const int s = blockIdx.x, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t SR = (int64_t)role_args(dev).S * role_args(dev).ring_total, SL = (int64_t)role_args(dev).S * role_args(dev).L;
    const bool count = kRings == kCounted && role_args(dev).disorder != 0;
    for (int i = 0; i < n_steps; ++i) {
        // states between the first and the last: tape entries, or the live copies in turn
        auto pos_at = [&](int k) { return tape_k >= 0 ? io.tape.pos + (tape_k + k) * SR : io.pos_mid[k & 1]; };
        auto seg_at = [&](int k) { return tape_k >= 0 ? io.tape.seg + (tape_k + k) * SL : io.seg_mid[k & 1]; };
        const bool first = i == 0, last = i == n_steps - 1;
        const StepAt at{first ? io.pos_in : pos_at(i), last ? io.pos_out : pos_at(i + 1), first ? io.pos_copy : nullptr,
                        first ? io.seg_in : seg_at(i), last ? io.seg_out : seg_at(i + 1),
                        first ? io.seg_copy : nullptr};
        // link tasks, longest rings first, the last wavefronts first (the first ones have the nodes)
        auto links = [&](auto &&f) {
            const Dev &d = role_args(dev);
            int task = kSoloWaves - 1 - w, done = 0, j0 = d.L;
#pragma unroll 1
            for (int c = kRingClasses - 1; c >= 0; --c) {
                const int n = d.lc_n[c], lanes = ring_lanes(c, d.g_link), lp = 6 - __builtin_ctz(lanes);
                const int tasks = (n + (1 << lp) - 1) >> lp;
                j0 -= n;
#pragma unroll 1
                for (; task < done + tasks; task += kSoloWaves) {
                    const int k = (task - done) << lp;
                    f(lanes, j0 + k, min(1 << lp, n - k));
                }
                done += tasks;
            }
        };
        const unsigned long long ts = stamp_begin(io.kstamp_node);
        if (count) {
            links([&](int lanes, int j, int n) { count_task(role_args(dev), at.pos_in, at.seg_in, lanes, s, j, n); });
            __syncthreads();
        }
        if (w < kSoloNodeWaves) {   // this wavefront's node task: the classes' tasks follow one another
            const Dev &d = role_args(dev);
            int k = w;
#pragma unroll 1
            for (int c = 0; c < 4; ++c) {
                const int per = 8 >> c, tasks = (d.nd_n[c] + per - 1) / per;
                if (k >= 0 && k < tasks)
                    node_task<kRings>(role_args(dev), at, io.tape, 8 << c, s, d.nd_begin[c] + k * per, min(per, d.nd_n[c] - k * per), t0 + i,
                              tape_k >= 0 ? tape_k + i : -1, inr + w * kWave, orc + w * kWave, crc + w * kWave, ckey + w * kWave);
                k = k < tasks ? -1 : k - tasks;
            }
        }
        stamp_end(io.kstamp_node, ts, s * kSoloWaves + w);
        const unsigned long long tl = stamp_begin(io.kstamp);
        links([&](int lanes, int j, int n) {
            link_task(role_args(dev), at, lanes, s, j, n, sample_bin(role_args(dev), t0 + i));
        });
        stamp_end(io.kstamp, tl, s * kSoloWaves + w);
        __syncthreads();
    }
    if (kRings == kCounted && home.pos) {   // a launch of its own for this copy took longer than a diamond's step
        const Dev &d = role_args(dev);
        const int64_t p0 = s * d.ring_total, l0 = (int64_t)s * d.L;
        for (int64_t i = threadIdx.x; i < d.ring_total; i += kSoloWaves * kWave) home.pos[p0 + i] = io.pos_out[p0 + i];
        for (int i = threadIdx.x; i < d.L; i += kSoloWaves * kWave) home.seg[l0 + i] = io.seg_out[l0 + i];
    }
}

// A descriptor into device memory, from the launch's own arguments: one small launch in a captured call, whose
// replays then do not depend on what the host holds by then.  Whether a placement put agents out of order is part
// of the state that a replay finds, not of the call that was captured.
__global__ void k_put_dev(Dev d, const int32_t *disorder, Dev *dst)
{
    if (threadIdx.x != 0) return;
    d.disorder = *disorder;
    *dst = d;
}

// Tape entry without an update (the state at the end of a replay window).
__global__ __launch_bounds__(256) void k_tape_snapshot(Dev d, const float *pos, const int4 *segs, Tape tp, int tape_k)
{
    const int lane = lane_id();
    const int seg = xcd_block() * kWavesPerBlock + (threadIdx.x >> 6);
    if (seg >= d.S * d.L) return;
    const int s = seg / d.L, j = seg - s * d.L;
    const int4 sg = segs[seg];
    const int n = sg.z - sg.x, cap = d.cap[j];
    const int64_t base = (int64_t)s * d.ring_total + d.ring_base[j];
    const int64_t tb = (int64_t)tape_k * d.S * d.ring_total + base;
    if (lane == 0) tp.seg[(int64_t)tape_k * d.S * d.L + seg] = sg;
    for (int r = lane; r < n; r += kWave) {
        const int slot = (sg.y + r) % cap;
        tp.pos[tb + slot] = pos[base + slot];
    }
}

// ---------------------------------------------------------------------------
// Reverse of step t (tape entry k holds time t, k+1 time t+1), per segment.
// The adjoint lives in a ring-parallel array: an agent keeps its ring slot
// while it is on a link, so a slot's entry is dL/dx of that slot's agent.
// Input: dL/dx(t+1) for slots live at t+1 (counts sampled at t+1 included).
// Output: dL/dx(t) for this link's slots live at t, plus the counts sampled at
// t; and the departure grafts of agents that entered this link during step t.
// Branches are recomputed from the taped time-t positions with the forward's
// exact float operations.
//   cap (SI-A eq. tg): dx_hat/dx' = 1 in both branches;
//   transfer (SI-B eq. transfer, SI-C): the entry position carries x_hat, so
//     a leaving head reads the adjoint at its entry slot (taped forward);
//   exit: total travel time falls by (x_hat - sg x_hat)/u of the last link;
//   free: x' = x + u dt; congested: x' = x_lead - dn/kappa; stopped: x' = x.
// Each agent has at most one follower (rank + lanes), so its adjoint is its own
// share plus what its follower hands on.  A lane group walks its ring front to
// back, kRevUnroll rounds of loads in flight: rank r takes its leader's position
// from the lanes of this round or the one before, and a round is finished (the
// followers' shares added, the result stored) when the next one is known; nothing
// goes through LDS.  The adjoint has two copies, read at t + 1 and written at t,
// so that the straight-through kernel can run beside it.
// kInit: dL/dx(T) at the final state (no step); that state is the handle's live
// one, whose rings name the agents.
// Bound: the chain link record -> taped counters -> positions and adjoints ->
// store, and the rounds that follow one another on a long ring.  So the launch
// needs few registers (7 wavefronts a SIMD) and few lanes a link rather than wide
// groups.  Against a kernel that staged each ring in LDS (16 lanes a link, 4
// wavefronts a SIMD at its largest): 1M-agent metro 15.3 -> 10.5 us a step, 16
// scenarios of 50k agents 21.7 -> 14.2, 6 x 6 lattice 5.4 -> 4.6; with the
// straight-through blocks, against two launches: 100-link network 20.0 -> 12.9,
// 64-candidate hub 30.6 -> 18.8.  Positions of 4 rounds are requested together
// and worked on in pairs: 2 or 4 alike in both cost 2-10 % of a gradient.
// ---------------------------------------------------------------------------
struct RevAt {
    const float *adj_in;   // dL/dx(t+1)
    float *adj_out;        // dL/dx(t)
};

// links [j0, j0 + count) of scenario s, one lane group of G lanes each
template <bool kInit>
__device__ __forceinline__ void reverse_task(const Dev &d, const Tape &tp, const RevAt &io, int G, int s, int j0, int count,
                                             int t, int tape_k)
{
    const Lanes g(G);
    const int gl = g.gl, gi = g.gbase >> __builtin_ctz(G);
    if (gi >= count) return;
    const int seg = s * d.L + j0 + gi;
    const int64_t SL = (int64_t)d.S * d.L;
    const int64_t ek = tape_k * SL + seg;          // tape entry of time t
    const int64_t ek1 = kInit ? ek : ek + SL;       // of time t+1 (the final state has none)
    // every per-segment value in one straight-line batch: link records, tape counters at t and
    // t+1, and the entry slots of the heads that left, read speculatively by the lanes below maxl
    // (a head that left has rank < lanes <= maxl <= G, so rank gl's is lane gl's)
    const LinkCf lc = d.lcf[seg];
    const RevCf rc = d.rcf[seg];
    const int4 ts = tp.seg[ek], ts1 = tp.seg[ek1];   // (head, head slot, tail, departures into this state)
    const int hk = ts.x, hm = ts.y, hk1 = ts1.x;
    const int depm = kInit ? 0 : ts1.w;             // entry orders of this step's departures
    const int ds_l = kInit ? -1 : tp.dst[ek * d.maxl + min(gl, d.maxl - 1)];
    const double gTs = d.gT ? d.gT[s] : 0.0;
    const int cap = lc.cap, ln = lc.lanes;
    const int n = min(ts.z - hk, cap);
    const int npass = kInit ? 0 : min(hk1 - hk, ln);
    // lane gl's head: its entry slot if it left during step t (-1: it left the network), else -2
    const int dsx = gl < npass ? ds_l : -2;
    const int64_t sR = (int64_t)s * d.ring_total, RTS = (int64_t)d.S * d.ring_total;
    const float *pos = tp.pos + (int64_t)tape_k * RTS + sR, *adj_in = io.adj_in + sR;
    float *adj_out = io.adj_out + sR;
    const float vf = lc.vf, sp = lc.sp, Lj = lc.L;
    const double dkap = rc.dkap;
    const float exit_adj = (float)(-gTs * rc.inv_u);
    const uint32_t first_off = (uint32_t)(lc.ring_base + hm) * 4u;
    auto off_of = [&](int r) { return first_off + 4u * (uint32_t)(hm + r >= cap ? r - cap : r); };
    int sb = -1;
    if (d.gQ && d.cbs > 0 && t > 0 && t % d.cbs == 0 && t / d.cbs <= d.nb) sb = t / d.cbs - 1;
    double gu = 0.0, gk = 0.0, gm = 0.0;
    const int lsrc = g.gbase + ((gl - ln) & (G - 1)), fsrc = g.gbase + ((gl + ln) & (G - 1));
    // rank r's adjoint: its own share and its follower's; on a sampling step (rare) the detectors' share, whose
    // values are read here, not held
    auto store = [&](int r, float x, float a) {
        if (sb >= 0) {
            const int d0 = lc.det & 0xffffff, nd = lc.det >> 24;
            const float sc = 5.0f / Lj;
            for (int k = 0; k < nd; ++k) {
                const int det = d.det_list[d0 + k];
                const int64_t qi = ((int64_t)s * d.D + det) * d.nb;
                const float gC = d.gQ[qi + sb] - (sb + 1 < d.nb ? d.gQ[qi + sb + 1] : 0.f);
                const float z = sc * (x - d.det_pos[det]);
                const float sg = 1.0f / (1.0f + expf(-z));
                a += gC * sc * sg * (1.0f - sg);
            }
        }
        if (r < n) at32(adj_out, off_of(r)) = a;
    };
    constexpr int U = kRevUnroll, P = 2;   // rounds of loads in flight; rounds worked on together
    float xprev = 0.f, keep = 0.f, push = 0.f;   // the last round: position, own share, the leader's share
    int last = 0;                                // its first rank
    for (int r0 = 0; r0 < n; r0 += U * G) {
        float xu[U], au[U];
        // rank r < G: the first round, where rank r is lane gl's head.  A head that left reads its adjoint
        // at the entry slot the tape names, or takes the exit term
        const bool left = r0 == 0 && dsx >= 0, gone = r0 == 0 && dsx == -1;
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const int r = r0 + q * G + gl;
            const bool in = r < n;
            xu[q] = in ? at32(pos, off_of(r)) : 0.f;
            if (q == 0 && left) au[q] = io.adj_in[dsx];
            else if (kInit) au[q] = in && d.gx ? d.gx[(int64_t)s * d.N + at32(d.ring_agent + sR, off_of(r))] : 0.f;
            else au[q] = in && !(q == 0 && gone) ? at32(adj_in, off_of(r)) : 0.f;
            if (q == 0 && gone) au[q] = exit_adj;
        }
        // admission-graft factor of a head that left on a token
        if (d.gm && left) gm += (double)au[0] * (double)tp.dstg[ek * d.maxl + gl];
#pragma unroll
        for (int p = 0; p < U; p += P) {
            if (r0 + p * G >= n) break;
            float *x = xu + p, *a = au + p, xl[P], kp[P], ps[P];
#pragma unroll
            for (int q = 0; q < P; ++q) xl[q] = __shfl(gl >= G - ln ? (q ? x[q ? q - 1 : 0] : xprev) : x[q], lsrc);
#pragma unroll
            for (int q = 0; q < P; ++q) {
                const float xf = x[q] + vf, xc = xl[q] - sp;
                const float cc = (x[q] > xc) ? x[q] : xc;
                // free, else stopped or congested; a rank past the ring has no share (a = 0)
                const bool free = kInit || (r0 + (p + q) * G + gl < ln) || xf <= cc, cong = !free && !(x[q] > xc);
                if (!kInit) {
                    gu += free ? d.dt * (double)a[q] : 0.0;
                    gk += cong ? dkap * (double)a[q] : 0.0;
                }
                kp[q] = cong ? 0.f : a[q];
                ps[q] = cong ? a[q] : 0.f;
            }
            // the follower of a round's last lanes is in the next round: round q - 1 is stored with round q known
#pragma unroll
            for (int q = 0; q < P; ++q) {
                const float pq = q ? ps[q ? q - 1 : 0] : push;
                const float fol = __shfl(gl >= ln ? pq : ps[q], fsrc);
                const float anew = (q ? kp[q ? q - 1 : 0] : keep) + fol;
                if (q > 0 || r0 + p > 0) store(r0 + (p + q - 1) * G + gl, q ? x[q ? q - 1 : 0] : xprev, anew);
            }
            last = r0 + (p + P - 1) * G;
            xprev = x[P - 1];
            keep = kp[P - 1];
            push = ps[P - 1];
        }
    }
    if (n > 0) {
        const float fol = __shfl(gl >= ln ? push : 0.f, fsrc);
        store(last + gl, xprev, keep + fol);
    }
    // departure grafts of the agents that entered this link during step t
    // an entrant of entry order e holds rank n + e at t+1 (the ring's free slots); the departures
    // among them are marked in the taped mask, so the agent and its adjoint are read together
    if (d.depg && gl < kMaxLanes && ((depm >> gl) & 1)) {
        const uint32_t o = off_of(n + gl);
        const int a = at32(tp.agent + (int64_t)(tape_k + 1) * RTS + sR, o);
        d.depg[(int64_t)s * d.N + a] = at32(adj_in, o) * rc.u;
    }
    g.sum2(gu, gk);
    if (d.gm) gm = g.sum(gm);
    // one non-returning atomic per accumulator: this group is the segment's only writer in the
    // launch, so the sum is the plain accumulator + contribution, without a read held in registers
    if (gl == 0 && !kInit) {
        const uint32_t off = (uint32_t)seg * 8u;   // every link has at least four ring slots: seg < 2^29
        unsafeAtomicAdd(&at32(d.gu, off), gu);
        unsafeAtomicAdd(&at32(d.gk, off), gk);
        if (d.gm) unsafeAtomicAdd(&at32(d.gm, off), gm);
    }
}

// ---------------------------------------------------------------------------
// Straight-through gradients of step t (SI-B), per node, in the launch of the
// reverse of step t, whose input dL/dx(t+1) they read too.  The
// hard route choices and merge winners of the forward are held; their relaxed
// weights (value 0, gradient of the softmax) enter the transfer update, so a
// candidate whose weight for its chosen link changes by dw changes the loss by
// G dw with
//   G = M adj(entry slot)            if it moved (entry position M + x - sg x),
//   G = -(M + x_hat) adj(own slot)   if it stayed on its in-link,
//   G = 0                            if an origin front stayed.
// Merge onto one link with k winners: k Plackett-Luce stages, stage s a
// softmax of (alpha_from l + g')/tau over the candidates ranked s and below
// (k = 1 is the single-winner merge of the text), l = 1 the candidate's
// relaxed weight of that link.  dL/d(merge utility) of a candidate is the sum
// over its stages of q (G - sum q G) / tau; alpha takes it directly and the
// route weight l takes alpha times it, which flows through the chosen link's
// softmax weight pi = softmax((V + g)/tau) into V_m = beta_m/c_m - theta r_m
// (r_m the link's free-flow time plus the shortest time to the destination).
// One lane group per (scenario, node) in the node classes of the forward;
// every accumulator has this node as its only writer (beta, cost: its
// out-links; alpha: its in-links; theta: its own entry), so the sums are
// deterministic.
//
// The softmax stages of one link share their sums.  With its candidates in key
// order y_0 >= y_1 >= ..., stage s has Z_s = sum_{r >= s} exp((y_r - y_s)/tau) =
// 1 + exp((y_{s+1} - y_s)/tau) Z_{s+1}, and likewise for the sum weighted with
// G: a linear recurrence down the order, taken for every link of the node at
// once by a segmented suffix scan over the lane group, one exp per candidate.
// (Each candidate summing every stage by itself took stages x candidates exps
// and divisions per lane: 138 us a launch at a 64-candidate node, 24 us on a
// 100-link network of small ones.)  The exponents are differences of
// neighbouring keys, never positive, so any tau is safe.  A node where no link
// is contested ends after the ranks.  The route softmax runs with a lane per
// out-link, not a loop over them in each lane: the double-precision logarithms
// and exponentials are then one copy of code (a wave's instruction fetch, cold
// at every launch, is a large part of its time).  138 -> 18.4 us a launch at the
// 64-candidate hub, 24.3 -> 12.8 us on the 100-link network.
// ---------------------------------------------------------------------------
struct SteLds {
    double *sy, *ty, *tg, *sd;   // keys, then 1/Z per place; keys in order; G in order, then its mean; dL/d(merge utility)
    int *sk, *sa;                // chosen out-link; agent, then the chosen out-link in order
};

__device__ __forceinline__ void ste_work(const Dev &d, const Tape &tp, const float *adj_in, const Lanes &g, int s, int v,
                                         int t, int tape_k, const SteLds &q)
{
    const int gl = g.gl, G = g.G;
    // every load goes out as soon as its address is known: node words and tables, the records of the
    // candidate's, the in-link's and the out-link's link, then the adjoint
    const int cnt = d.node_cnt[v];
    const int64_t rbase = d.route_base[v];
    const int cb = d.cbase[v];
    const int jin = max(d.in_pad[(int64_t)v * d.max_in + min(gl, d.max_in - 1)], 0);
    const int joff = d.in_loff[(int64_t)v * d.max_in + min(gl, d.max_in - 1)];
    const int deg = cnt & 0xff, dego = (cnt >> 8) & 0xff, norg = (cnt >> 16) & 0xff;
    const int nc = ((cnt >> 24) & 0xff) + norg;
    const int64_t sL = (int64_t)s * d.L, sR = (int64_t)s * d.ring_total;
    const int4 rc = gl < nc ? tp.ste[((int64_t)tape_k * d.S + s) * d.n_cand + cb + gl] : make_int4(-1, 0, -1, -1);
    int D = 4;   // lanes per choosing candidate of the route softmax, lane m its out-link m
    while (D < dego) D <<= 1;
    const int m = gl & (D - 1);
    const int om = max(d.out_pad[(int64_t)v * d.max_out + min(m, d.max_out - 1)], 0);
    const bool cand = rc.x >= 0;
    const int total = g.count(cand);
    if (total < 2) return;   // a lone candidate has weight 1 in every softmax
    const int ag = rc.x, argk = cand ? rc.y & 0xff : -1, kst = (rc.y >> 8) & 0xff, moved = (rc.y >> 16) & 1;
    const int from = rc.z, loc = rc.w;
    const double tau = d.tau;
    const uint64_t seed = d.seed[s];
    const bool has = cand && loc >= 0;
    const float adj = has ? adj_in[sR + loc] : 0.f;
    const float xh = has && !moved ? tp.pos[(int64_t)(tape_k + 1) * d.S * d.ring_total + sR + loc] : 0.f;
    const LinkNd &fl = d.lnd[sL + max(from, 0)];
    const float alf = fl.alpha;
    const int ftl = fl.tail;
    const int row = cand ? d.agent_didx[ag] : 0;
    const LinkNd &ol = d.lnd[sL + om];
    const double outil = ol.util;
    const int ohead = ol.head, jlanes = d.lnd[sL + jin].lanes;
    const int ftail = from >= 0 ? ftl : -1;
    const double al = from >= 0 ? (double)alf : 1.0;
    double y = 0.0;
    if (cand) {
        uint32_t w[4];
        draw4(seed, ag, t, 1, 0, w);
        y = al + gumbel_of(w[0]);
    }
    q.sy[gl] = y;
    q.sk[gl] = argk;
    q.sa[gl] = ag;
    wave_lds_sync();
    // place in the merge order of its target (key descending, agent id on ties), group size, and the
    // candidates of earlier targets
    int rho = 0, n = 1, base = 0;
    constexpr int kCk = 4;
    for (int e0 = 0; e0 < nc; e0 += kCk)
#pragma unroll
    for (int k = 0; k < kCk; ++k) {
        const int e = (e0 + k) & (G - 1), k2 = q.sk[e], a2 = q.sa[e];
        const double y2 = q.sy[e];
        const bool in = cand & (e0 + k < nc) & (k2 >= 0), same = in & (k2 == argk) & (e != gl);
        base += in & (k2 < argk);
        n += same;
        rho += same & ((y2 > y) | ((y2 == y) & (a2 < ag)));
    }
    const bool contest = cand && n >= 2;
    if (g.count(contest) == 0) return;   // every candidate is alone on its link: nothing to share
    const double Gc = !has ? 0.0 : (moved ? d.big_m * (double)adj : -(d.big_m + (double)xh) * (double)adj);
    wave_lds_sync();
    if (cand) {
        q.ty[base + rho] = y;
        q.tg[base + rho] = Gc;
        q.sa[base + rho] = argk;
    }
    wave_lds_sync();
    {   // place gl of the order: sums over the places at and behind it on its link
        const int me = gl < total ? q.sa[gl] : -1;
        const bool more = gl + 1 < total && q.sa[min(gl + 1, G - 1)] == me;
        const double yi = gl < total ? q.ty[gl] : 0.0, yn = more ? q.ty[min(gl + 1, G - 1)] : yi;
        double z = 1.0, zg = gl < total ? q.tg[gl] : 0.0, a = more ? exp((yn - yi) / tau) : 0.0;
        for (int o = 1; o < G; o <<= 1) {   // a lane whose link ends within o places has a = 0 by then
            const int up = min(gl + o, G - 1);
            const double z2 = g.from(z, up), g2 = g.from(zg, up), a2 = g.from(a, up);
            z += a != 0.0 ? a * z2 : 0.0;
            zg += a != 0.0 ? a * g2 : 0.0;
            a = a != 0.0 ? a * a2 : 0.0;
        }
        wave_lds_sync();
        q.sy[gl] = 1.0 / z;
        q.tg[gl] = zg / z;
        wave_lds_sync();
    }
    double dVp = 0.0;
    if (contest) {
        const int K = min(min(n, kst), rho + 1);
        for (int st = 0; st < K; ++st) {
            const int p = base + st;
            dVp += exp((y - q.ty[p]) / tau) * q.sy[p] / tau * (Gc - q.tg[p]);
        }
    }
    q.sd[gl] = dVp;
    wave_lds_sync();
    if (gl < deg) {   // alpha of in-link gl: its candidate lanes in order
        double a = 0.0;
        bool any = false;
        for (int r = 0; r < jlanes; ++r) { a += q.sd[joff + r]; any |= q.sk[joff + r] >= 0; }
        if (any) unsafeAtomicAdd(&d.galpha[sL + jin], a);   // this group's own entry: no read to wait for
    }
    const double gam = al * dVp;
    if (g.count(gam != 0.0) == 0) return;
    // route choice: softmax of (V + g)/tau over the admissible out-links, then dV_m per out-link.  The
    // group splits into parts of D >= out-degree lanes, each taking one choosing candidate at a time.
    // The hard choice is the argmax of the same scores, so the chosen link's is the softmax's maximum.
    const bool on = cand && gam != 0.0;
    const unsigned long long om_on = g.mask(on);
    const int n_on = __popcll(om_on);
    if (on) q.sa[__popcll(om_on & ((1ull << gl) - 1ull))] = gl;
    wave_lds_sync();
    double mys = 0.0, th = 0.0;
    for (int c0 = 0; c0 < n_on; c0 += G / D) {
        const int c = c0 + gl / D;
        const bool act = c < n_on;
        const int src = act ? q.sa[c] : gl;
        const int cag = g.from(ag, src), cch = g.from(argk, src), crow = g.from(row, src);
        const int cfrom = g.from(from, src), ctail = g.from(ftail, src);
        const double cgam = g.from(gam, src);
        const bool in = act & (m < dego);
        const double rk = in ? d.route[rbase + (int64_t)crow * dego + m] : INFINITY;
        uint32_t w[4];
        draw4(seed, cag, t, 0, m >> 2, w);
        const uint32_t wk = (m & 2) ? ((m & 1) ? w[3] : w[2]) : ((m & 1) ? w[1] : w[0]);
        const bool ok = in & !((!d.allow_uturn) & (cfrom >= 0) & (ohead == ctail)) & (rk < INFINITY);
        const double sc = outil - d.theta * (ok ? rk : 0.0) + gumbel_of(wk);
        const double top = g.from(sc, (gl & ~(D - 1)) + cch);
        const double e = ok ? exp((sc - top) / tau) : 0.0;
        double Z = e;
        for (int o = 1; o < D; o <<= 1) Z += __shfl_xor(Z, o);
        if (ok) {
            const double dv = cgam / tau / Z * ((m == cch ? 1.0 : 0.0) - e / Z);
            mys += dv;
            th -= rk * dv;
        }
    }
    for (int o = D; o < G; o <<= 1) mys += __shfl_xor(mys, o);
    if (gl < dego && mys != 0.0) {
        const double c = (double)d.cost[sL + om], b = (double)d.beta[sL + om];
        unsafeAtomicAdd(&d.gbeta[sL + om], mys / c);
        unsafeAtomicAdd(&d.gcost[sL + om], -(b / (c * c) * mys));
    }
    th = g.sum(th);
    if (gl == 0) unsafeAtomicAdd(&d.gth[(int64_t)s * d.Nn + v], th);
}

// ---------------------------------------------------------------------------
// One launch per reverse step: block roles for each ring class's links (64 / lanes to a wavefront) and, with
// straight-through gradients, for each node class's nodes, which run first (their chains are the longest).
// Each role is remapped so that neighbours share an XCD.  A window's steps in one launch of one workgroup, as
// the forward step has them for small networks, gain nothing here: 10.7 ms for 600 steps of a 6 x 6 lattice
// with its gradient, 10.3 with a launch per step.
// ---------------------------------------------------------------------------
// A launch's block roles: the node classes from the widest (only with ste), then the ring classes from the
// longest.  They go as kernel arguments, so that a block knows its work without a chain of descriptor reads.
struct RevRoles {
    struct Role { int block, blocks, first, n; } role[8];   // first block, blocks; first node or link, their number
};

enum { kRevInit, kRevStep, kRevStepSte };
template <int kMode>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kMode == kRevStepSte ? 4 : 7)))
void k_reverse(const Dev *dev, Tape tp, RevIo io, RevRoles roles, unsigned long long *kstamp, int g_rev, int t, int tape_k)
{
    constexpr bool STE = kMode == kRevStepSte;
    const unsigned long long t0 = stamp_begin(kstamp);
    const Dev &d = role_args(dev);
    const RevAt at{io.adj[(t + 1) & 1], io.adj[t & 1]};
    int c = STE ? 0 : 4;
    RevRoles::Role R = roles.role[c];
#pragma unroll
    for (int k = c + 1; k < 8; ++k)
        if ((int)blockIdx.x >= roles.role[k].block) { R = roles.role[k]; c = k; }
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wb = xcd_remap((int)blockIdx.x - R.block, R.blocks) * kWavesPerBlock + w;
    if (STE && c < 4) {
        __shared__ double sy[256], ty[256], tg[256], sd[256];
        __shared__ int sk[256], sa[256];
        const Lanes g(64 >> c);
        const int item = wb * (1 << c) + (g.gbase >> (6 - c));
        if (item < d.S * R.n) {
            const int s = scenario_of(item, R.n, d.S), o = w * kWave + g.gbase;
            ste_work(d, tp, at.adj_in, g, s, R.first + item - s * R.n, t, tape_k,
                     SteLds{sy + o, ty + o, tg + o, sd + o, sk + o, sa + o});
        }
    } else {   // a wavefront's links lie in one scenario
        const int lanes = ring_lanes(7 - c, g_rev), lg = __builtin_ctz(lanes), per = kWave >> lg;
        const int tasks = (R.n + per - 1) >> (6 - lg);
        const int s = scenario_of(wb, max(tasks, 1), d.S), j = (wb - s * tasks) * per;
        if (s < d.S && j < R.n) 
            reverse_task<kMode == kRevInit>(d, tp, at, lanes, s, R.first + j, min(per, R.n - j), t, tape_k);
    }
    stamp_end(kstamp, t0, (int64_t)blockIdx.x * kWavesPerBlock + w);
}

// theta gradient of each scenario: the per-node parts summed in node order by one wavefront
__global__ __launch_bounds__(64) void k_theta_sum(Dev d, float *out)
{
    const int s = blockIdx.x;
    double a = 0.0;
    for (int v = lane_id(); v < d.Nn; v += kWave) a += d.gth[(int64_t)s * d.Nn + v];
    a = wave_sum_d(a);
    if (lane_id() == 0) out[s] = (float)a;
}

// dL/d rates[s, o, b] = sum over departed agents of origin o of
// depg * overlap(bin b, [0, t*)) / rate(release bin): the departure-time
// graft (the entry position moves by u * (change of release time)).
// One wavefront per (scenario, origin), lane = bin, agents in queue order.
__global__ __launch_bounds__(256) void k_rate_grad(Dev d, float *g)
{
    const int lane = lane_id();
    const int wid = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
    if (wid >= d.S * d.O) return;
    const int s = wid / d.O, o = wid - s * d.O;
    const int nbins = d.n_rate_bins;
    const int qb = d.q_off[o], qn = d.q_off[o + 1] - qb;
    const int64_t sN = (int64_t)s * d.N;
    const float *rates = d.rates + ((int64_t)s * d.O + o) * nbins;
    // lanes take the queue's agents 64 at a time; per bin, a fixed-order wave sum (deterministic)
    double accb = 0.0;   // lane b < nbins (in its round of 64 bins) holds bin b's total
    for (int b0 = 0; b0 < nbins; b0 += kWave) {
        accb = 0.0;
        for (int k0 = 0; k0 < qn; k0 += kWave) {
            const int k = k0 + lane;
            double dg = 0.0, rt = 1.0, ts = 0.0;
            if (k < qn) {
                const int a = d.q_list[qb + k];
                if (d.dep_t[sN + a] >= 0) {
                    ts = d.tstar[sN + a];
                    const int rb = min(nbins - 1, max(0, (int)floor((double)d.rel_t[sN + a] * d.dt / d.rate_bin_s)));
                    dg = (double)d.depg[sN + a];
                    rt = (double)rates[rb];
                }
            }
            for (int bb = 0; bb < kWave && b0 + bb < nbins; ++bb) {
                const int b = b0 + bb;
                const double ov = fmin((b + 1) * d.rate_bin_s, ts) - b * d.rate_bin_s;
                double c = (dg != 0.0 && ov > 0) ? dg * ov / rt : 0.0;
                for (int off = 32; off > 0; off >>= 1) c += __shfl_xor(c, off);
                if (lane == bb) accb += c;
            }
        }
        if (b0 + lane < nbins) g[((int64_t)s * d.O + o) * nbins + b0 + lane] = (float)accb;
    }
}

// Derived per-(scenario, link) constants.
__global__ void k_derive(Dev d, const float *cap_mult, const float *capacity, const float *beta,
                         const float *cost, double *acc, LinkNd *lnd, LinkCf *lcf, RevCf *rcf)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)d.S * d.L) return;
    const int j = (int)(i % d.L);
    acc[i] = (double)cap_mult[i] * (double)capacity[j] * (double)d.lanes[j] * d.dt;
    LinkNd c;
    c.util = (double)beta[i] / (double)cost[i];
    c.alpha = d.alpha[i];
    c.head = d.head[j];
    c.tail = d.tail[j];
    c.lanes = d.lanes[j];
    lnd[i] = c;
    LinkCf f;
    f.vf = __fmul_rn(d.u[i], (float)d.dt);
    f.sp = __fdiv_rn((float)d.platoon, d.kappa[i]);
    f.L = d.length[j];
    f.thr = d.thr[j];
    f.cap = d.cap[j];
    f.lanes = d.lanes[j];
    f.ring_base = d.ring_base[j];
    f.det = d.det_off[j] | ((d.det_off[j + 1] - d.det_off[j]) << 24);
    lcf[i] = f;
    RevCf rv;
    const double kd = (double)d.kappa[i];
    rv.dkap = (double)d.platoon / (kd * kd);
    rv.inv_u = 1.0 / (double)d.u[i];
    rv.u = d.u[i];
    rv.pad = 0;
    rcf[i] = rv;
}

// The checkpoint's arrays in one launch: 16-byte chunks grid-strided over each array, then its
// byte tail (all arrays start on 256-byte boundaries).
__global__ __launch_bounds__(256) void k_copy_multi(CopyJobs jobs)
{
    const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t nth = (uint64_t)gridDim.x * blockDim.x;
    for (int k = 0; k < jobs.n; ++k) {
        const uint4 *src = static_cast<const uint4 *>(jobs.job[k].src);
        uint4 *dst = static_cast<uint4 *>(jobs.job[k].dst);
        const uint64_t nv = jobs.job[k].bytes / 16, rem = jobs.job[k].bytes - nv * 16;
        for (uint64_t i = tid; i < nv; i += nth) dst[i] = src[i];
        if (tid < rem)
            static_cast<char *>(jobs.job[k].dst)[nv * 16 + tid] =
                static_cast<const char *>(jobs.job[k].src)[nv * 16 + tid];
    }
}

// The same for arrays set to a word each (bytes of the word alike where an array is not whole words).
__global__ __launch_bounds__(256) void k_fill_multi(FillJobs jobs)
{
    const uint64_t tid = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const uint64_t nth = (uint64_t)gridDim.x * blockDim.x;
    for (int k = 0; k < jobs.n; ++k) {
        uint4 *dst = static_cast<uint4 *>(jobs.job[k].dst);
        const uint32_t w = jobs.job[k].word;
        const uint64_t nv = jobs.job[k].bytes / 16, rem = jobs.job[k].bytes - nv * 16;
        for (uint64_t i = tid; i < nv; i += nth) dst[i] = make_uint4(w, w, w, w);
        if (tid < rem) static_cast<char *>(jobs.job[k].dst)[nv * 16 + tid] = (char)w;
    }
}

// Total travel time and vehicle-steps per scenario: agent-steps spent queued or on the network, (exit step or T) -
// release step summed over released agents, and those on the network, (exit step or T) - departure step over
// departed ones.  Integer sums, exact in int64 whatever the order; each block adds its own with one atomic, and
// k_ttt_final scales by dt.
__global__ __launch_bounds__(256) void k_ttt(Dev d, int T, unsigned long long *acc)
{
    const int s = blockIdx.y;
    const int64_t sN = (int64_t)s * d.N;
    long long tt = 0, vs = 0;
    for (int i = blockIdx.x * 256 + threadIdx.x; i < d.N; i += gridDim.x * 256) {
        const uint8_t st = d.status[sN + i];
        if (st == AG_WAIT) continue;
        const int e = (st == AG_EXITED) ? d.exit_t[sN + i] : T;
        tt += e - d.rel_t[sN + i];
        if (st != AG_QUEUED) vs += e - (d.dep_t[sN + i] >= 0 ? d.dep_t[sN + i] : 0);  // placed agents: from t = 0
    }
    for (int o = 32; o > 0; o >>= 1) { tt += __shfl_xor(tt, o); vs += __shfl_xor(vs, o); }
    __shared__ long long p[2][kWavesPerBlock];
    if ((threadIdx.x & 63) == 0) { p[0][threadIdx.x >> 6] = tt; p[1][threadIdx.x >> 6] = vs; }
    __syncthreads();
    if (threadIdx.x == 0) {
        long long a = 0, b = 0;
        for (int w = 0; w < kWavesPerBlock; ++w) { a += p[0][w]; b += p[1][w]; }
        atomicAdd(&acc[2 * s], (unsigned long long)a);
        atomicAdd(&acc[2 * s + 1], (unsigned long long)b);
    }
}

// Route table of a network of up to kRouteNodes nodes, one workgroup a destination: shortest free-flow times by
// relaxing every node from its out-links in LDS until nothing changes, then the destination's row of every node.
// A time is the minimum over paths of the sum w + (rest) taken from the destination outwards, whatever order
// the relaxations come in: rounding keeps the order of sums, so Dijkstra on the host finds the same doubles.
// A round relaxes the nodes with an out-link to one that got nearer since their last turn (a bit per node).  A
// value that another wavefront is improving at the time may be seen old or new (8-byte LDS accesses are whole):
// the improvement marks the node for the next round.  At most a round per node; after `rounds` without an end the
// workgroup leaves its rows unwritten and says so.
// Bound: rounds, each a few dependent reads of L2 and LDS.  1.2 ms a table, averaged over eight networks of
// 1,000 to 35,000 links and 16 to 1,024 destinations, 5.1 ms when every round relaxes every node; on the host,
// the 35,000-link one took half a second of 8 threads, and its table of 290 MB was copied over.
__global__ __launch_bounds__(1024) void k_route(int Nn, int nd, const int32_t *out_off, const OutEdge *edge,
                                                const int32_t *in_off, const int32_t *in_tail, const int32_t *dest,
                                                int rounds, int32_t *gave_up, double *route)
{
    extern __shared__ double time_to[];   // [Nn], then two sets of a bit per node: this round's and the next one's
    __shared__ int changed[2];
    const int words = (Nn + 31) >> 5;
    uint32_t *turn = reinterpret_cast<uint32_t *>(time_to + Nn);
    const int k = blockIdx.x, me = dest[k];
    auto get = [&](int v) { return __hip_atomic_load(&time_to[v], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
    auto mark = [&](int v, uint32_t *set) {   // v got nearer: the nodes with a link to it
        for (int j = in_off[v]; j < in_off[v + 1]; ++j) atomicOr(&set[in_tail[j] >> 5], 1u << (in_tail[j] & 31));
    };
    for (int v = threadIdx.x; v < Nn; v += 1024) time_to[v] = v == me ? 0.0 : INFINITY;
    for (int i = threadIdx.x; i < 2 * words; i += 1024) turn[i] = 0u;
    if (threadIdx.x < 2) changed[threadIdx.x] = 0;
    __syncthreads();
    if (threadIdx.x == 0) mark(me, turn);
    for (int it = 0;; ++it) {
        uint32_t *cur = turn + (it & 1) * words, *nxt = turn + (~it & 1) * words;
        __syncthreads();
        bool any = false;
        for (int v = threadIdx.x; v < Nn; v += 1024) {
            if (!((cur[v >> 5] >> (v & 31)) & 1u)) continue;
            const int b = out_off[v], e = out_off[v + 1];
            const double now = get(v);
            double best = now;
            for (int j = b; j < e; ++j) best = fmin(best, edge[j].time + get(edge[j].head));
            if (best < now) {
                __hip_atomic_store(&time_to[v], best, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                mark(v, nxt);
                any = true;
            }
        }
        if (any) changed[it & 1] = 1;
        __syncthreads();
        if (changed[it & 1] == 0) break;
        if (it >= rounds) {
            if (threadIdx.x == 0) *gave_up = 1;
            return;
        }
        for (int i = threadIdx.x; i < words; i += 1024) cur[i] = 0u;
        if (threadIdx.x == 0) changed[~it & 1] = 0;
    }
    __syncthreads();
    for (int v = threadIdx.x; v < Nn; v += 1024) {
        const int b = out_off[v], dg = out_off[v + 1] - b;
        double *row = route + (int64_t)nd * b + (int64_t)k * dg;
        for (int j = 0; j < dg; ++j) row[j] = edge[b + j].time + time_to[edge[b + j].head];
    }
}

__global__ void k_zero_u64(unsigned long long *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0ull;
}
__global__ void k_ttt_final(int S, double dt, const unsigned long long *acc, double *out, int64_t *vsteps)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= S) return;
    out[s] = (double)(long long)acc[2 * s] * dt;
    if (vsteps) vsteps[s] = (int64_t)(long long)acc[2 * s + 1];
}

// Interval counts from cumulative samples.
__global__ void k_counts(Dev d, float *out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)d.S * d.D * d.nb) return;
    const int b = (int)(i % d.nb);
    out[i] = (float)(d.cum[i] - (b > 0 ? d.cum[i - 1] : 0));
}

// dst[s, caller link] = src[s, internal link], double -> float
__global__ void k_gather_links(const double *src, const int32_t *linv, float *dst, int S, int L)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)S * L) return;
    const int64_t s = i / L, jo = i - s * L;
    dst[i] = (float)src[s * L + linv[jo]];
}

__global__ void k_d2f(const double *src, float *dst, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = (float)src[i];
}

__global__ void k_philox(int n, const uint32_t *ctr, const uint32_t *key, uint32_t *out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t c[4] = {ctr[4 * i], ctr[4 * i + 1], ctr[4 * i + 2], ctr[4 * i + 3]};
    philox4x32_10(c, key[2 * i], key[2 * i + 1]);
    for (int k = 0; k < 4; ++k) out[4 * i + k] = c[k];
}


// ---------------------------------------------------------------------------
// Segmented sort: keys (segment, position, sequence) -> permutation in
// segment order, position descending, sequence ascending, input index
// ascending.  A counting pass by segment (histogram, scan, scatter) places
// every key in its segment; then each segment is ranked by comparison: the
// 96-bit keys (flipped position bits, sequence, index) are all different, so a
// key's place is the number of keys below it.  Segments up to kSortMax keys.
//
// Who ranks a segment follows its length.  A link of the simulator holds tens
// of agents, so a wavefront takes two segments of at most 32 keys side by side
// (one LDS read per compared key serves both), or one of at most 64; the
// rivals' keys come from LDS, 16 bytes a read.  Longer ones are taken by the
// whole workgroup: n / 256 keys a lane against n up to kSortRank, and a bitonic
// network in LDS above, where n^2 comparisons cost more than its
// log2(n)^2 / 2 barriers.  1,000,000 keys in 35,000 segments: 39 us (24 passes of
// a 4-bit radix sort with a counter column per thread took 5,290 us); the whole
// sort 152 us, most of it the two passes of a million scattered atomics (45 and
// 58 us, 22 and 17 per ns).
// ---------------------------------------------------------------------------
constexpr int kSortMax = 2048;
constexpr int kSortRank = 512;                        // block-ranked up to here, bitonic above
constexpr int kSortThreads = 256;
constexpr int kSortSegs = 2 * kWavesPerBlock;         // segments per workgroup, two per wavefront
constexpr int kSortKeys = 2;                          // keys per thread of the scatter
constexpr int kScanTile = 4096;                       // counters per workgroup of the scan

// clears the counters and the overflow flag in one launch (no memset node)
__global__ __launch_bounds__(256) void k_seg_clear(int32_t *cnt, int64_t n, int32_t *err)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) cnt[i] = 0;
    if (i == 0) *err = 0;
}

__global__ __launch_bounds__(256) void k_seg_hist(int n, const int32_t *seg, int32_t *cnt)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) atomicAdd(&cnt[seg[i]], 1);
}

// sum of v over the workgroup (256 lanes), and the exclusive prefix of the lane's v
__device__ __forceinline__ int32_t block_prefix(int32_t v, int32_t *wsum, int32_t &total)
{
    const int lane = lane_id(), w = threadIdx.x >> 6;
    int32_t x = v;
    for (int o = 1; o < kWave; o <<= 1) {
        const int32_t y = __shfl_up(x, o);
        if (lane >= o) x += y;
    }
    if (lane == kWave - 1) wsum[w] = x;
    __syncthreads();
    int32_t before = 0;
    total = 0;
    for (int k = 0; k < kWavesPerBlock; ++k) { before += k < w ? wsum[k] : 0; total += wsum[k]; }
    __syncthreads();
    return before + x - v;
}

// exclusive scan of n_seg counts -> off[0..n_seg] and the cursors: the tiles' sums, then per tile
// the sums before it and the scan within it (one workgroup over all counters took 77 us at 35,000)
__global__ __launch_bounds__(256) void k_seg_tile_sum(int n_seg, const int32_t *cnt, int32_t *part)
{
    __shared__ int32_t wsum[kWavesPerBlock];
    const int b = blockIdx.x * kScanTile;
    int32_t sum = 0, total;
    for (int q = 0; q < kScanTile / 256; ++q) {
        const int i = b + q * 256 + threadIdx.x;
        sum += i < n_seg ? cnt[i] : 0;
    }
    block_prefix(sum, wsum, total);
    if (threadIdx.x == 0) part[blockIdx.x] = total;
}

__global__ __launch_bounds__(256) void k_seg_scan(int n_seg, const int32_t *cnt, const int32_t *part, int32_t *off,
                                                  int32_t *cursor)
{
    __shared__ int32_t wsum[kWavesPerBlock];
    int32_t sum = 0, run;
    for (int i = threadIdx.x; i < (int)blockIdx.x; i += 256) sum += part[i];
    block_prefix(sum, wsum, run);
    const int b = blockIdx.x * kScanTile;
    int32_t c[kScanTile / 256];
#pragma unroll
    for (int q = 0; q < kScanTile / 256; ++q) {
        const int i = b + q * 256 + threadIdx.x;
        c[q] = i < n_seg ? cnt[i] : 0;
    }
#pragma unroll
    for (int q = 0; q < kScanTile / 256; ++q) {
        const int i = b + q * 256 + threadIdx.x;
        int32_t total;
        const int32_t e = run + block_prefix(c[q], wsum, total);
        if (i < n_seg) { off[i] = e; cursor[i] = e; }
        if (i == n_seg - 1) off[n_seg] = e + c[q];
        run += total;
    }
}

__global__ __launch_bounds__(256) void k_seg_scatter(int n, const int32_t *seg, int32_t *cursor, int32_t *out)
{
    const int64_t i0 = (int64_t)blockIdx.x * (256 * kSortKeys) + threadIdx.x;
    int32_t s[kSortKeys], p[kSortKeys];
#pragma unroll
    for (int q = 0; q < kSortKeys; ++q) s[q] = i0 + q * 256 < n ? seg[i0 + q * 256] : -1;
#pragma unroll
    for (int q = 0; q < kSortKeys; ++q) p[q] = s[q] >= 0 ? atomicAdd(&cursor[s[q]], 1) : 0;
#pragma unroll
    for (int q = 0; q < kSortKeys; ++q)
        if (s[q] >= 0) out[p[q]] = (int32_t)(i0 + q * 256);
}

__device__ __forceinline__ uint32_t desc_float_key(float x)
{
    uint32_t u = __float_as_uint(x == 0.0f ? 0.0f : x);
    u = (u & 0x80000000u) ? ~u : (u | 0x80000000u);  // ascending order of x
    return ~u;                                        // descending
}

// key of input index idx: (high word: position, then sequence; low word: the index itself)
struct alignas(16) SortKey { uint64_t k; uint32_t idx, pad; };
__device__ __forceinline__ SortKey sort_key(int32_t idx, const float *pos, const int32_t *seq)
{
    return SortKey{((uint64_t)desc_float_key(pos[idx]) << 32) | ((uint32_t)seq[idx] ^ 0x80000000u), (uint32_t)idx, 0u};
}
__device__ __forceinline__ int key_below(const SortKey &a, const SortKey &b)
{
    return (a.k < b.k) | ((a.k == b.k) & (a.idx < b.idx));
}

__global__ __launch_bounds__(kSortThreads) void k_seg_sort(int n_seg, const int32_t *off, const float *pos,
                                                           const int32_t *seq, int32_t *perm, int32_t *err)
{
    __shared__ SortKey key[kSortMax];
    const int tid = threadIdx.x, lane = lane_id(), w = tid >> 6;
    const int s0 = blockIdx.x * kSortSegs, sw = s0 + 2 * w;
    {
        // this wavefront's two segments; offsets past the last segment read as empty
        const int o0 = off[min(sw, n_seg)], o1 = off[min(sw + 1, n_seg)], o2 = off[min(sw + 2, n_seg)];
        SortKey *buf = key + w * kWave;
        const bool two = o1 - o0 <= 32 && o2 - o1 <= 32;
        for (int h = 0; h < (two ? 1 : 2); ++h) {
            // two: lanes 0-31 the first segment, 32-63 the second; else a whole wavefront per segment
            const int half = two ? lane >> 5 : h, l = two ? lane & 31 : lane;
            const int b = half ? o1 : o0, n = (half ? o2 : o1) - b;
            const bool on = n > 1 && n <= kWave;
            SortKey me{0, 0, 0};
            if (on && l < n) me = sort_key(perm[b + l], pos, seq);
            buf[lane] = me;
            wave_lds_sync();
            const SortKey *seg = buf + (two ? half * 32 : 0);
            int rank = 0;
            const int m = two ? max(o1 - o0, o2 - o1) : (on ? n : 0);
#pragma unroll 4
            for (int e = 0; e < m; ++e) rank += (e < n) & key_below(seg[e], me);
            if (on && l < n) perm[b + rank] = (int32_t)me.idx;
            wave_lds_sync();
        }
    }
    // the workgroup's longer segments, one after another: every gridDim-th one, so that neighbours go to different
    // workgroups.  Their offsets are read together, a lane each.
    const int64_t sl = blockIdx.x + (int64_t)min(lane, kSortSegs - 1) * gridDim.x;
    const int bl = off[min(sl, (int64_t)n_seg)], nl = off[min(sl + 1, (int64_t)n_seg)] - bl;
    for (int g = 0; g < kSortSegs; ++g) {
        const int b = __builtin_amdgcn_readlane(bl, g), n = __builtin_amdgcn_readlane(nl, g);
        if (n <= kWave) continue;
        if (n > kSortMax) { if (tid == 0) atomicOr(err, 1); continue; }
        __syncthreads();
        if (n <= kSortRank) {
            SortKey me[kSortRank / kSortThreads];
            int rank[kSortRank / kSortThreads];
#pragma unroll
            for (int q = 0; q < kSortRank / kSortThreads; ++q) {
                const int i = tid + q * kSortThreads;
                rank[q] = 0;
                me[q] = i < n ? sort_key(perm[b + i], pos, seq) : SortKey{0, 0, 0};
                if (i < n) key[i] = me[q];
            }
            __syncthreads();
#pragma unroll 4
            for (int e = 0; e < n; ++e) {
                const SortKey o = key[e];
#pragma unroll
                for (int q = 0; q < kSortRank / kSortThreads; ++q) rank[q] += key_below(o, me[q]);
            }
#pragma unroll
            for (int q = 0; q < kSortRank / kSortThreads; ++q)
                if (tid + q * kSortThreads < n) perm[b + rank[q]] = (int32_t)me[q].idx;
        } else {
            const int P = n <= 1024 ? 1024 : 2048;
            for (int i = tid; i < P; i += kSortThreads)   // padding sorts behind every key
                key[i] = i < n ? sort_key(perm[b + i], pos, seq) : SortKey{~0ull, 0xffffffffu, 0u};
            __syncthreads();
            for (int k = 2; k <= P; k <<= 1)
                for (int j = k >> 1; j > 0; j >>= 1) {
                    for (int p = tid; p < P / 2; p += kSortThreads) {
                        const int i = ((p & ~(j - 1)) << 1) | (p & (j - 1)), x = i | j;
                        const SortKey a = key[i], c = key[x];
                        if (key_below(c, a) == ((i & k) == 0)) { key[i] = c; key[x] = a; }
                    }
                    __syncthreads();
                }
            for (int i = tid; i < n; i += kSortThreads) perm[b + i] = (int32_t)key[i].idx;
        }
        __syncthreads();
    }
}

// Workgroups of the segment sort: eight segments each, or for few segments one each, which may all be long (8 segments
// of 2,000 keys in one workgroup took 837 us).
static unsigned sort_blocks(int n_seg)
{
    return (unsigned)std::max<int64_t>(((int64_t)n_seg + kSortSegs - 1) / kSortSegs, std::min(n_seg, 1024));
}
static int scan_tiles(int n_seg) { return (int)(((int64_t)n_seg + kScanTile - 1) / kScanTile); }
int64_t segsort_scratch_words(int n_seg) { return 2 * ((int64_t)n_seg + 1) + scan_tiles(n_seg) + 1; }

// The sort proper on caller-provided scratch: cnt and cursor [n_seg + 1],
// part [scan_tiles(n_seg)], err [1].  The scratch is cleared with a fill kernel
// (no memset node), and nothing here waits for the device.
static int enqueue_segsort(int n, int n_seg, const int32_t *seg, const float *pos, const int32_t *seq,
                           int32_t *perm, int32_t *seg_off, int32_t *cnt, int32_t *cursor, int32_t *part, int32_t *err,
                           hipStream_t st)
{
    const int64_t nc = (int64_t)n_seg + 1;
    const unsigned kb = (unsigned)(((int64_t)n + 256 * kSortKeys - 1) / (256 * kSortKeys));
    hipLaunchKernelGGL(k_seg_clear, dim3((unsigned)((nc + 255) / 256)), dim3(256), 0, st, cnt, nc, err);
    if (n > 0) hipLaunchKernelGGL(k_seg_hist, dim3((unsigned)(((int64_t)n + 255) / 256)), dim3(256), 0, st, n, seg, cnt);
    if (scan_tiles(n_seg) > 1)   // a single tile has no tiles before it
        hipLaunchKernelGGL(k_seg_tile_sum, dim3(scan_tiles(n_seg)), dim3(256), 0, st, n_seg, cnt, part);
    hipLaunchKernelGGL(k_seg_scan, dim3(scan_tiles(n_seg)), dim3(256), 0, st, n_seg, cnt, part, seg_off, cursor);
    if (n > 0) {
        hipLaunchKernelGGL(k_seg_scatter, dim3(kb), dim3(256), 0, st, n, seg, cursor, perm);
        hipLaunchKernelGGL(k_seg_sort, dim3(sort_blocks(n_seg)), dim3(kSortThreads), 0, st, n_seg, seg_off, pos, seq, perm, err);
    }
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

static int read_sort_flag(const int32_t *err, hipStream_t st)
{
    int32_t e = 0;
    if (hipMemcpyAsync(&e, err, 4, hipMemcpyDeviceToHost, st) != hipSuccess) return -1;
    if (hipStreamSynchronize(st) != hipSuccess) return -1;
    return e ? 1 : 0;
}

int launch_segsort(int n, int n_seg, const int32_t *seg, const float *pos, const int32_t *seq, int32_t *perm,
                   int32_t *seg_off, int32_t *scratch, hipStream_t st)
{
    int32_t *cnt = scratch, *cursor = cnt + ((int64_t)n_seg + 1), *part = cursor + ((int64_t)n_seg + 1);
    int32_t *err = part + scan_tiles(n_seg);
    if (enqueue_segsort(n, n_seg, seg, pos, seq, perm, seg_off, cnt, cursor, part, err, st) != 0) return -1;
    return read_sort_flag(err, st);
}

// ---------------------------------------------------------------------------
// Allocation-free segmented sort: its counters live in one fixed device
// array per GPU instead of a per-call allocation.  The array's name is only
// a host-side stand-in; its device address comes from hipGetSymbolAddress,
// taken once per device with that device current (segsort_scratch_init,
// called when a handle is created) and used for every launch and copy.
// ---------------------------------------------------------------------------
static __device__ __align__(256) int32_t
    scratch[2 * (kNoAllocMaxSegments + 1) + 64 + kNoAllocMaxSegments / kScanTile];

namespace {
std::mutex g_scratch_mu;
int32_t *g_scratch_ptr[kMaxDevices] = {};
}

int segsort_scratch_init(int device)
{
    if (device < 0 || device >= kMaxDevices) return -1;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_ptr[device]) return 0;
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess || cur != device) return -1;
    int32_t *p = nullptr;
    if (hipGetSymbolAddress((void **)&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return -1;
    g_scratch_ptr[device] = p;
    return 0;
}

int launch_segsort_noalloc(int device, int n, int n_seg, const int32_t *seg, const float *pos, const int32_t *seq,
                           int32_t *perm, int32_t *seg_off, int32_t *status, hipStream_t st)
{
    if (n_seg < 1 || n_seg > kNoAllocMaxSegments) return -2;
    int32_t *base = nullptr;
    {
        std::lock_guard<std::mutex> lk(g_scratch_mu);
        if (device >= 0 && device < kMaxDevices) base = g_scratch_ptr[device];
    }
    if (!base) return -1;
    int32_t *cnt = base, *cursor = base + (n_seg + 1), *flag = base + 2 * (kNoAllocMaxSegments + 1), *part = flag + 64;
    int32_t *err = status ? status : flag;
    if (enqueue_segsort(n, n_seg, seg, pos, seq, perm, seg_off, cnt, cursor, part, err, st) != 0) return -1;
    return status ? 0 : read_sort_flag(err, st);
}

// ---------------------------------------------------------------------------
// Optimisation loop (calibration and control, Methods "Optimization"): the
// count loss with its cotangent, and the AdamW update of one parameter group.
// ---------------------------------------------------------------------------

// One workgroup.  kind 0: mean over the n = det x nb counts of (q - y)^2,
// cotangent 2 (q - y) / n.  kind 1: (sum over the bins of detector det of q
// - target)^2, cotangent 2 (sum - target) on those bins, 0 elsewhere.  Fixed
// reduction order, so the loss is reproducible.
__global__ __launch_bounds__(1024) void k_count_loss(int n, int nb, const float *q, const float *y, int kind,
                                                      int det, double target, double *loss, float *gq)
{
    __shared__ double part[1024];
    const int tid = threadIdx.x;
    double acc = 0.0;
    if (kind == 0) {
        for (int i = tid; i < n; i += 1024) {
            const double e = (double)q[i] - (double)y[i];
            acc += e * e;
            gq[i] = (float)(2.0 * e / (double)n);
        }
    } else {
        for (int i = tid; i < n; i += 1024) gq[i] = 0.0f;
        if (tid < nb) acc = (double)q[(int64_t)det * nb + tid];
    }
    part[tid] = acc;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (tid < o) part[tid] += part[tid + o];
        __syncthreads();
    }
    if (kind == 0) {
        if (tid == 0) *loss = n > 0 ? part[0] / (double)n : 0.0;
    } else {
        const double e = part[0] - target;
        if (tid == 0) *loss = e * e;
        if (tid < nb) gq[(int64_t)det * nb + tid] = (float)(2.0 * e);
    }
}

// AdamW (Loshchilov and Hutter, decoupled weight decay) on float parameters
// in the coordinates x = (p - x0) / sc (x0 = 0, sc = 1: the parameters
// themselves), update t >= 1 with the gradient gx = g sc:
// m <- b1 m + (1 - b1) gx, v <- b2 v + (1 - b2) gx^2,
// x <- x - lr (m / (1 - b1^t) / (sqrt(v / (1 - b2^t)) + eps) + wd x),
// p = x0 + sc x, then the box [lo, min(hi, hi_vec[i])].  Arithmetic in double.
__global__ void k_adamw(int64_t n, float *p, const float *g, float *m, float *v, int t, double lr, double b1,
                        double b2, double eps, double wd, double x0, double sc, double lo, double hi,
                        const float *hi_vec)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double gi = (double)g[i] * sc;
    const double mi = b1 * (double)m[i] + (1.0 - b1) * gi;
    const double vi = b2 * (double)v[i] + (1.0 - b2) * gi * gi;
    m[i] = (float)mi;
    v[i] = (float)vi;
    const double mh = mi / (1.0 - pow(b1, (double)t));
    const double vh = vi / (1.0 - pow(b2, (double)t));
    double x = ((double)p[i] - x0) / sc;
    x = x - lr * (mh / (sqrt(vh) + eps) + wd * x);
    double y = x0 + sc * x;
    double top = hi;
    if (hi_vec) top = fmin(top, (double)hi_vec[i]);
    y = fmin(fmax(y, lo), top);
    p[i] = (float)y;
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
void launch_count_loss(int n, int nb, const float *q, const float *y, int kind, int det, double target,
                       double *loss, float *gq, hipStream_t st)
{
    hipLaunchKernelGGL(k_count_loss, dim3(1), dim3(1024), 0, st, n, nb, q, y, kind, det, target, loss, gq);
}

void launch_adamw(int64_t n, float *p, const float *g, float *m, float *v, int t, double lr, double b1, double b2,
                  double eps, double wd, double x0, double sc, double lo, double hi, const float *hi_vec,
                  hipStream_t st)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_adamw, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, n, p, g, m, v, t, lr, b1, b2,
                       eps, wd, x0, sc, lo, hi, hi_vec);
}
static inline int blocks_for(int64_t waves) { return (int)((waves + kWavesPerBlock - 1) / kWavesPerBlock); }

// one wavefront per launch record (offset, waves): first start and last end over its waves
__global__ __launch_bounds__(256) void k_stamp_reduce(const int64_t *off, const int32_t *waves, int n,
                                                      const unsigned long long *st, unsigned long long *out)
{
    const int r = (int)blockIdx.x * kWavesPerBlock + ((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
    if (r >= n) return;
    const unsigned long long *p = st + 2 * off[r];
    unsigned long long lo = ~0ull, hi = 0ull;
    for (int w = lane; w < waves[r]; w += 64) {
        lo = min(lo, p[2 * w]);
        hi = max(hi, p[2 * w + 1]);
    }
    for (int o = 32; o > 0; o >>= 1) {
        lo = min(lo, (unsigned long long)__shfl_xor(lo, o));
        hi = max(hi, (unsigned long long)__shfl_xor(hi, o));
    }
    if (lane == 0) { out[2 * r] = lo; out[2 * r + 1] = hi; }
}
void launch_stamp_reduce(const int64_t *off, const int32_t *waves, int n, const unsigned long long *st,
                         unsigned long long *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_stamp_reduce, dim3((n + kWavesPerBlock - 1) / kWavesPerBlock), dim3(256), 0, s, off, waves,
                       n, st, out);
}

static StepRoles step_roles(const Dev &d, int rows)
{
    StepRoles r{};
    constexpr int LW = kStepWaves - 1;
    int slot = 0;
    for (int c = 0; c < 4; ++c) {
        const int n = d.nd_n[3 - c], tasks = (n + (1 << c) - 1) >> c;
        r.node[c] = {slot, d.nd_begin[3 - c], n};
        slot += (tasks + rows - 1) / rows * rows;
    }
    r.blocks = slot;
    int link = d.L;
    slot = 0;
    for (int c = 0; c < 4; ++c) {
        const int n = d.lc_n[3 - c], per = kWave / ring_lanes(3 - c, d.g_link), tasks = (n + per - 1) / per;
        link -= n;
        r.link[c] = {slot, link, n};
        slot += ((tasks + rows - 1) / rows + LW - 1) / LW * LW * rows;
    }
    r.blocks = std::max(r.blocks, slot / LW);
    return r;
}
// A launch's roles, and whether they are packed (kXcd = 0).  Rows keep neighbouring tasks of a scenario on one XCD.  So
// do packed tasks where the number of scenarios is a multiple of 8 (block b of scenario s lies on XCD s % 8): 16
// scenarios of 50k agents with their adjoint 60.5 ms packed, 61.1 in rows.  With other numbers rows win (45x45 lattice, 15
// scenarios, a step: 14.6 us, packed 17.6; 14x14, 257: 24.2, 26.2) unless a fifth of them is padding and their workgroups
// exceed what the chip holds at once (diamond, 4,095 scenarios: 28.2, packed 16.2; 4x4 38.6, 27.6; 6x6 64.6, 63.8).
static bool packed_roles(const Dev &d, StepRoles &r)
{
    r = step_roles(d, 8);
    if (d.S == 1) return false;
    constexpr int kAtOnce = 256 * 4 * 6 / kStepWaves;   // workgroups: 256 CUs, 4 SIMDs, 6 wavefronts
    const StepRoles p = step_roles(d, 1);
    const bool packed = d.S % 8 == 0 || ((int64_t)d.S * r.blocks > kAtOnce && 4 * r.blocks > 5 * p.blocks);
    if (packed) r = p;
    return packed;
}
void step_waves(const Dev &d, bool solo, int64_t *link, int64_t *node)
{
    StepRoles r;
    (void)packed_roles(d, r);
    const int64_t blocks = (int64_t)d.S * r.blocks;
    *link = solo ? (int64_t)d.S * kSoloWaves : blocks * (kStepWaves - 1);
    *node = solo ? (int64_t)d.S * kSoloWaves : blocks;
}
void launch_step(const Dev &d, const Dev *dev, const StepIo &io, const HomeIo &home, bool solo, bool captured, int t, int n_steps,
                 int tape_k, hipStream_t st)
{
    auto go_solo = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(d.S), dim3(kSoloWaves * kWave), 0, st, dev, io, home, t, n_steps, tape_k);
    };
    if (solo && !captured && !d.disorder) return go_solo(k_step_solo<kOrdered>);
    if (solo) return go_solo(k_step_solo<kCounted>);
    StepRoles r;
    const bool packed = packed_roles(d, r);
    const dim3 grid(d.S * r.blocks), block(kStepWaves * kWave);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, st, dev, io, r, d.g_link, t, tape_k);
    };
    if (captured || !d.disorder) return packed ? go(k_step<kScan, 0>) : go(k_step<kScan, 3>);
    hipLaunchKernelGGL(packed ? k_ring_counts<0> : k_ring_counts<3>, grid, block, 0, st, dev, io.pos_in, io.seg_in, r, d.g_link);
    packed ? go(k_step<kCounted, 0>) : go(k_step<kCounted, 3>);
}
template <class Jobs>
static int jobs_blocks(const Jobs &jobs)
{
    uint64_t total = 0;
    for (int k = 0; k < jobs.n; ++k) total += jobs.job[k].bytes / 16;
    return (int)std::max<uint64_t>(1, std::min<uint64_t>((total + 255) / 256, 2048));
}
void launch_copy_multi(const CopyJobs &jobs, hipStream_t st)
{
    hipLaunchKernelGGL(k_copy_multi, dim3(jobs_blocks(jobs)), dim3(256), 0, st, jobs);
}
void launch_fill_multi(const FillJobs &jobs, hipStream_t st)
{
    hipLaunchKernelGGL(k_fill_multi, dim3(jobs_blocks(jobs)), dim3(256), 0, st, jobs);
}
static int reverse_roles(const Dev &d, bool ste, RevRoles &r)
{
    int block = 0, link = d.L;
    for (int c = 0; c < 8; ++c) {
        const int lanes = c < 4 ? 64 >> c : ring_lanes(7 - c, d.g_rev), per = kWave / lanes;
        const int n = c < 4 ? (ste ? d.nd_n[3 - c] : 0) : d.lc_n[7 - c];
        const int tasks = c < 4 ? (d.S * n + per - 1) / per : d.S * ((n + per - 1) / per);
        const int blocks = ((tasks + kWavesPerBlock - 1) / kWavesPerBlock + 7) & ~7;   // whole rows of XCDs
        if (c >= 4) link -= n;
        r.role[c] = {block, blocks, c < 4 ? d.nd_begin[3 - c] : link, n};
        block += blocks;
    }
    return block;
}
int reverse_waves(const Dev &d, bool ste)
{
    RevRoles r;
    return reverse_roles(d, ste, r) * kWavesPerBlock;
}

void launch_reverse(const Dev &d, const Dev *dev, const Tape &tp, const RevIo &io, unsigned long long *kstamp, bool ste, int t,
                    int tape_k, int init, hipStream_t st)
{
    RevRoles r;
    const dim3 grid(reverse_roles(d, ste, r)), block(256);
    auto go = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, block, 0, st, dev, tp, io, r, kstamp, d.g_rev, t, tape_k);
    };
    if (init) go(k_reverse<kRevInit>);
    else if (ste) go(k_reverse<kRevStepSte>);
    else go(k_reverse<kRevStep>);
}
void launch_put_dev(const Dev &d, const int32_t *disorder, Dev *dst, hipStream_t st)
{
    hipLaunchKernelGGL(k_put_dev, dim3(1), dim3(kWave), 0, st, d, disorder, dst);
}
void launch_tape_snapshot(const Dev &d, const float *pos, const int4 *seg, const Tape &tp, int tape_k, hipStream_t st)
{
    hipLaunchKernelGGL(k_tape_snapshot, dim3(blocks_for((int64_t)d.S * d.L)), dim3(256), 0, st, d, pos, seg, tp, tape_k);
}
hipError_t launch_route(int Nn, int nd, const int32_t *out_off, const OutEdge *edge, const int32_t *in_off,
                        const int32_t *in_tail, const int32_t *dest, int rounds, int32_t *gave_up, double *route, hipStream_t st)
{
    static_assert(route_lds(kRouteNodes) + 8 <= 160 * 1024, "the times have to fit the LDS");
    const hipError_t e =
        hipFuncSetAttribute((const void *)k_route, hipFuncAttributeMaxDynamicSharedMemorySize, route_lds(kRouteNodes));
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_route, dim3(nd), dim3(1024), route_lds(Nn), st, Nn, nd, out_off, edge, in_off, in_tail, dest, rounds,
                       gave_up, route);
    return hipGetLastError();
}
void launch_theta_sum(const Dev &d, float *out, hipStream_t st)
{
    hipLaunchKernelGGL(k_theta_sum, dim3(d.S), dim3(64), 0, st, d, out);
}
void launch_rate_grad(const Dev &d, float *g, hipStream_t st)
{
    if ((int64_t)d.S * d.O == 0) return;
    hipLaunchKernelGGL(k_rate_grad, dim3(blocks_for((int64_t)d.S * d.O)), dim3(256), 0, st, d, g);
}
void launch_derive(const Dev &d, const float *cap_mult, const float *capacity, const float *beta,
                   const float *cost, double *acc, LinkNd *lnd, LinkCf *lcf, RevCf *rcf, hipStream_t st)
{
    const int64_t n = (int64_t)d.S * d.L;
    hipLaunchKernelGGL(k_derive, dim3((int)((n + 255) / 256)), dim3(256), 0, st, d, cap_mult, capacity, beta, cost,
                       acc, lnd, lcf, rcf);
}
void launch_ttt(const Dev &d, int T, double *out, int64_t *vsteps, unsigned long long *acc, hipStream_t st)
{
    // acc: 2 x S zeroed here with a fill kernel (no memset node, so the sequence can sit in a graph)
    hipLaunchKernelGGL(k_zero_u64, dim3((2 * d.S + 255) / 256), dim3(256), 0, st, acc, 2 * d.S);
    const int nb = std::max(1, std::min(1024, (d.N + 2047) / 2048));
    hipLaunchKernelGGL(k_ttt, dim3(nb, d.S), dim3(256), 0, st, d, T, acc);
    hipLaunchKernelGGL(k_ttt_final, dim3((d.S + 255) / 256), dim3(256), 0, st, d.S, d.dt, acc, out, vsteps);
}
void launch_counts(const Dev &d, float *out, hipStream_t st)
{
    const int64_t n = (int64_t)d.S * d.D * d.nb;
    if (n == 0) return;
    hipLaunchKernelGGL(k_counts, dim3((int)((n + 255) / 256)), dim3(256), 0, st, d, out);
}
void launch_gather_links(const double *src, const int32_t *linv, float *dst, int S, int L, hipStream_t st)
{
    const int64_t n = (int64_t)S * L;
    if (n == 0) return;
    hipLaunchKernelGGL(k_gather_links, dim3((int)((n + 255) / 256)), dim3(256), 0, st, src, linv, dst, S, L);
}
void launch_d2f(const double *src, float *dst, int64_t n, hipStream_t st)
{
    if (n == 0) return;
    hipLaunchKernelGGL(k_d2f, dim3((int)((n + 255) / 256)), dim3(256), 0, st, src, dst, n);
}
__global__ void k_gumbel_fast(int n, const uint32_t *w, float *out)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = gumbel_fast(w[i]);
}
void launch_gumbel_fast(int n, const uint32_t *w, float *out, hipStream_t st)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_gumbel_fast, dim3((n + 255) / 256), dim3(256), 0, st, n, w, out);
}
void launch_philox(int n, const uint32_t *ctr, const uint32_t *key, uint32_t *out, hipStream_t st)
{
    if (n <= 0) return;
    hipLaunchKernelGGL(k_philox, dim3((n + 255) / 256), dim3(256), 0, st, n, ctr, key, out);
}

}  // namespace sim

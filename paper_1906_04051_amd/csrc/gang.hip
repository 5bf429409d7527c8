// Whole deflated GMRES(m) solves in one persistent launch.
//
// A gang of K workgroups (one per compute unit, all on the chip together) owns
// a system: workgroup `me` owns a contiguous range of RW sliced
// positions, one to four rows a thread.  The Krylov basis of those rows lives in the
// workgroup's LDS (columns that do not fit there in global memory, read only
// by their owner), so the two Gram-Schmidt sweeps of a step touch no HBM.
// The arithmetic is the two-sweep CGS2 with lagged normalisation of
// krylov.hip (arXiv 1906.04051, Sec. 3.2-3.3: eqs. krylov-basis, hessenberg,
// arg, res, new_sol, relative, precond2); Hessenberg, rotations and restart
// decisions are computed redundantly by every workgroup from the same sums in
// the same order, so no workgroup waits for a serial kernel.
//
// Why: below about 300,000 rows two steps of the kernel-per-phase engine are a
// dozen dependent launches of 4-10 us each, whatever the size, against a few us
// of memory traffic.  Here a step is three rendezvous of the gang (two without
// a deflation basis).  us per step, gang / engine: 4,225 rows, 16 columns, m =
// 30, 12.6 / 27.3; 30,276 rows, no columns, 9.6 / 18.3; 66,049 rows, 64 columns,
// m = 50, 19.1 / 32.9; where the engine wins, see gang_basis_limit.
//
// Rendezvous: each workgroup stores its epoch in its own flag word and polls
// all K words (one coalesced load per try); no read-modify-write, no central
// counter.  Everything that crosses workgroups (the SpMV input vector, the
// iterate, partial sums, flags) is stored and loaded with relaxed agent-scope
// atomics, which go past the per-die L2s, and every wave waits for its stores
// (vmcnt(0)) before its workgroup's flag is set; nothing else is shared, so no
// cache is written back or invalidated and the matrix stays in L2.
//
// All of a gang has to be on the chip.  It is an ordinary launch on the plan's
// stream (a cooperative one would take one of the process's four hardware
// queues for good: 25 systems continued on their own streams then took 1,080 ms
// instead of 745), so the host keeps the gangs of this process apart: a launch
// holds as many compute units of every die as its workgroups need there
// (GangPlace), and one that does not fit beside the others waits for them.
// Kernels of other streams or processes that hold compute units are not in that
// account, so every wait in the kernel ends: the first rendezvous, which shows
// that all of the gang is there, gives up after start_ticks (10 ms by default),
// any later one, which only a fault or a preempted queue can hold up, after
// wait_ticks (2 s); a wait longer than 1 ms also ends when the abort word shows
// that another workgroup has given up.  The launch then ends with that word set,
// and the host repeats the solve on the kernel-per-phase engine and leaves the
// gang out of the next solves.
//
// Adaptive deflation (MODE == kGangAdapt; adapt.hip): M^{-1} changes at every
// restart and its update needs the basis, so a launch runs one cycle.  Within
// it U^T x rides on the exchange that already carries the second projection's
// sums (no further rendezvous) and A U C U^T x is added behind the SpMV; the
// basis goes to memory once, at the end, for the Ritz step's kernels.  Ritz
// steps included, gang / engine (one step per pair of sweeps there): a Newton
// solve of Bratu 20^3 (about 263 steps, m = 50) 8.8 / 18.0 ms; 66,049 rows, m =
// 50, up to 22 columns, 30 cycles: 25.8 / 57.7 us a step; 361,201 rows, m = 30,
// 8 cycles: 47.6 / 76.4.
#include "internal.hpp"

#include <chrono>
#include <condition_variable>
#include <mutex>

namespace gm {

constexpr int kGN = 512;                      // threads per workgroup
constexpr int kGW = kGN / kWave;              // wavefronts

// Pointers with their address space spelled out: accesses that could go to
// either memory must not be merged into flat ones.
#define GM_LDS __attribute__((address_space(3)))
#define GM_GLB __attribute__((address_space(1)))

template <typename T>
__device__ __forceinline__ T ld_ag(const T* p) {
    return __hip_atomic_load((const GM_GLB T*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void st_ag(T* p, T v) {
    __hip_atomic_store((GM_GLB T*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Stored form of a basis entry (half precision as the native type, which may
// live in any address space).
template <typename T>
struct Stored {
    using type = T;
};
template <>
struct Stored<__half> {
    using type = _Float16;
};

// Values that are the same in every lane, in a scalar register: the branches
// and loops they control are then scalar too.
__device__ __forceinline__ int uni(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ bool unib(bool x) { return __builtin_amdgcn_readfirstlane((int)x) != 0; }
__device__ __forceinline__ int64_t uni64(int64_t x) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)x);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(x >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double unid(double x) { return __longlong_as_double(uni64(__double_as_longlong(x))); }

// ------------------------------------------------------------ wave reductions
// Sums of eight values over the wavefront: halving exchanges (32, 16, 8 lanes)
// leave lane l with the sum of value ((l >> 3) & 1) + 2 ((l >> 4) & 1) +
// 4 (l >> 5): ten exchanges instead of 48.
template <typename T>
__device__ __forceinline__ T gsum8(const T (&v)[8], int ln) {
    T r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = swap_add<true>(v[i], v[i + 4]);
    const T q0 = swap_add<false>(r[0], r[2]);
    const T q1 = swap_add<false>(r[1], r[3]);
    const bool up = (ln & 8) != 0;
    T z = (up ? q1 : q0) + gdpp<0x128>(up ? q0 : q1);   // row_ror:8
    z += gdpp<0xB1>(z);
    z += gdpp<0x4E>(z);
    z += gdpp<0x141>(z);
    return z;
}
// The same for sixteen values (17 exchanges): lane l holds value
// gsum16_col(l).
template <typename T>
__device__ __forceinline__ T gsum16(const T (&v)[16], int ln) {
    T r[8], q[4], y[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = swap_add<true>(v[i], v[i + 8]);
#pragma unroll
    for (int i = 0; i < 4; ++i) q[i] = swap_add<false>(r[i], r[i + 4]);
    const bool b8 = (ln & 8) != 0, b4 = (ln & 4) != 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) y[i] = (b8 ? q[i + 2] : q[i]) + gdpp<0x128>(b8 ? q[i] : q[i + 2]);   // row_ror:8
    T z = (b4 ? y[1] : y[0]) + gdpp<0x141>(b4 ? y[0] : y[1]);
    z += gdpp<0xB1>(z);
    z += gdpp<0x4E>(z);
    return z;
}
__device__ __forceinline__ int gsum16_col(int ln) {
    return 8 * (ln >> 5) + 4 * ((ln >> 4) & 1) + 2 * ((ln >> 3) & 1) + ((ln >> 2) & 1);
}
__device__ __forceinline__ int gsum8_col(int ln) {
    return ((ln >> 3) & 1) + 2 * ((ln >> 4) & 1) + 4 * (ln >> 5);
}

// ------------------------------------------------------------------ rendezvous
// Every workgroup's flag (and its row of partial sums) has cache lines of its
// own: with the flags side by side a rendezvous of 207 workgroups took 2.65
// us, on lines of their own 1.38 us (34: 1.29 and 1.18; trees of flags 1.9 and
// 1.6, one counter 3.1 and 1.1, in a loop of nothing else).
constexpr int kFlagW = kGangFlagWords;

// All of the workgroup's shared stores are in memory; its flag shows `epoch`.
__device__ __forceinline__ void gang_arrive(int K, int me, unsigned* flags, unsigned epoch) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (K > 1 && threadIdx.x == 0) st_ag(flags + me * kFlagW, epoch);
}
// A wait of `waited` ticks has to end; nothing is loaded before it has lasted
// h.look ticks.  kWaitSystem: members of a batch's gang that have no part in its
// system wait for the others, who end it or give up.
constexpr int kWaitSum = 0, kWaitStart = 1, kWaitSystem = 2;
__device__ __forceinline__ bool gang_expired(long long waited, const GangHot& h, const GangArgs& a, int kind) {
    return waited > h.look && ((kind != kWaitSystem && waited > (kind == kWaitStart ? a.start_ticks : a.wait_ticks)) ||
                               ld_ag(a.abortw) != 0);
}
// Waits until every member of the gang shows `epoch`; false (in every thread)
// after a timeout.
__device__ __forceinline__ bool gang_wait(int K, const unsigned* flags, unsigned epoch, int* s_abort,
                                          const GangHot& h, const GangArgs& a, int kind) {
    if (K == 1) return true;
    if ((int)threadIdx.x < K) {
        const unsigned* f = flags + threadIdx.x * kFlagW;
        const long long t0 = wall_clock64();
        while ((int)(ld_ag(f) - epoch) < 0) {
            if (gang_expired(wall_clock64() - t0, h, a, kind)) {
                *s_abort = 1;
                break;
            }
        }
    }
    __syncthreads();
    return !uni(*s_abort);
}
#define GANG_ARRIVE() gang_arrive(K, me, flags, ++epoch)
#define GANG_FAIL()                           \
    do {                                      \
        if (tid == 0) st_ag(a.abortw, 1u);    \
        return;                               \
    } while (0)
#define GANG_WAIT_FOR(K_, kind)                                                   \
    do {                                                                          \
        if (!gang_wait(K_, flags, epoch, s_abort, h, a, kind)) GANG_FAIL();       \
    } while (0)
#define GANG_WAIT() GANG_WAIT_FOR(K, epoch == 1 ? kWaitStart : kWaitSum)

// Sums travel without flags: an entry that is not there yet holds a
// signalling NaN, which no arithmetic result is (operations return quiet
// ones), and readers load until it is gone.  That saves the wait for the
// data's acknowledgement and one round trip per rendezvous.
constexpr unsigned long long kEmpty = 0x7FF4C0DEC0DEC0DEull;
__device__ __forceinline__ unsigned long long ld_bits(const double* p) {
    return ld_ag(reinterpret_cast<const unsigned long long*>(p));
}
__device__ __forceinline__ void st_empty(double* p) {
    st_ag(reinterpret_cast<unsigned long long*>(p), kEmpty);
}

// Sums of up to 64 columns over the K members' rows (stride ps) of partial
// sums, once every entry is there: lane = column, so a load takes one member's
// row -- two or four rows where the columns fit half or a quarter of the lanes
// (W = 32, 16).  The waves take members in turn, eight loads in flight each;
// the wave's sums go to redrow.
template <int W>
__device__ __forceinline__ void gang_rows(int nc, const double* part, int ps, int K, int wv, int ln,
                                          double* redrow, int* s_abort, const GangHot& h, const GangArgs& a) {
    constexpr int MPL = kWave / W, U = 8;
    const int col = min(ln & (W - 1), nc - 1), sub = ln / W;
    double t = 0;
    for (int i0 = wv * MPL; i0 < K; i0 += U * kGW * MPL) {
        const int i = i0 + sub;
        unsigned long long v[U];
        long long t0 = 0;
        for (;;) {
            bool wait = false;
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] = ld_bits(part + min(i + u * kGW * MPL, K - 1) * ps + col);
#pragma unroll
            for (int u = 0; u < U; ++u) wait |= v[u] == kEmpty;
            if (!__any(wait)) break;
            const long long now = wall_clock64();
            if (t0 == 0) t0 = now;
            if (gang_expired(now - t0, h, a, kWaitSum)) {
                *s_abort = 1;
                break;
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) t += i + u * kGW * MPL < K ? __longlong_as_double((long long)v[u]) : 0.0;
    }
    if (MPL >= 4) t = swap_add<false>(t, t);
    if (MPL >= 2) t = swap_add<true>(t, t);
    if (ln < W) redrow[ln] = t;
}

// ---------------------------------------------------------------------- kernel
// The small state has a fixed place in LDS (immediate addresses); the
// Hessenberg (packed columns), the cached rows of E^{-1} and the basis follow
// in the dynamic part.
constexpr int kGangSingle = 0, kGangBatch = 1, kGangAdapt = 2;
constexpr int kMP = (kMaxM + 9) & ~7;   // slots per column array
constexpr int kAU = 24;                 // adaptive deflation columns (kAdaptMax rounded up)
constexpr int kZS = 64;                 // Z columns summed per round
__host__ __device__ inline int gang_hraw(int m) { return ((m * (m + 3) / 2) + 7) & ~7; }

template <typename AT, typename VT, typename WT, typename BT, typename ACC, int RPT, int WF, int MODE>
__global__ __launch_bounds__(kGN) void k_gang(GangHot h, const GangArgs* ac) {
    // Arguments of the cold paths are read from memory where they are used
    // (they would otherwise fill the scalar registers of the step loop).
    const GangArgs& a = *ac;
    constexpr bool BATCH = MODE == kGangBatch, ADAPT = MODE == kGangAdapt;
    extern __shared__ double dyn[];
    __shared__ double cs[kMP], sn[kMP], gl[kMP], h1[kMP], h2[kMP], ds[kMP + kAU];
    __shared__ ACC c1[kMP], c2[kMP];           // coefficients of the sweeps
    __shared__ double red[kGW][kMP + 8 + kAU]; // per-wave dots, norm at kMP, U dots from kMP + 8
    __shared__ double grow[kGW][2 * kWave];    // per-wave sums over the members
    __shared__ double zred[kGW][kZS];          // per-wave Z^T sums
    __shared__ double tv[kMaxR], sv[kMaxR];    // t = Z^T u, s = E^{-1} t
    __shared__ double su[ADAPT ? kAU : 1];     // C U^T x
    __shared__ int zl[kMaxR], al[kMaxR];       // own Z columns; columns whose s is needed
    __shared__ int rng[kMaxR];                 // members [lo, hi) touching each column
    __shared__ unsigned bits[32];              // 8 words Z, 8 words A Z
    __shared__ int si[8];                      // abort, nz, na, estimate met, system, multi, breakdown
    const int tid = threadIdx.x, wv = uni(threadIdx.x / kWave), ln = tid & (kWave - 1);
    const int m = h.m;
    constexpr bool kHalf = sizeof(VT) == 2;
    using ST = typename Stored<VT>::type;
    double* Hr = dyn;                          // unrotated Hessenberg, column j at j(j+3)/2
    double* El = dyn + gang_hraw(m);           // ecap bytes
    GM_LDS ST* Vl = (GM_LDS ST*)((char*)El + h.ecap);
    int* s_abort = si;

    // ---- gang membership
    const int me = BATCH ? uni(a.wg_member[blockIdx.x]) : (int)blockIdx.x;
    const int Kg = BATCH ? uni(a.wg_size[blockIdx.x]) : h.K;
    const int first = (int)blockIdx.x - me;
    unsigned epoch = 0;
    // Published systems alternate between two words: a member without a part
    // in a system may read its word while the leader publishes the next one.
    int turn = 0;
    unsigned* flags = h.flags + first * kFlagW;
    const int ps = gang_ps(m + 2 + (ADAPT ? kAU : 0)), ts = gang_ps(h.Rmax);   // row strides
    // Exchange e of the gang uses slot e % 3: a workgroup empties its row of
    // exchange e once it has collected e + 1 (which everyone published after
    // collecting e), and waits for that store before it publishes e + 2, so a
    // reader of e + 3 never meets the old entry.  The Z^T rows alternate
    // between two slots in the same way, with at least two exchanges between.
    double* ring = h.part + (int64_t)first * 3 * ps;
    double* trow = h.tpart + (int64_t)first * 2 * ts;
    int slot = 0, pslot = 0, pcount = 0, tslot = 0, tpend = -1;
    unsigned* bmap = a.bmap + (int64_t)first * 8;

    // A workgroup that finds a place after the others have given up leaves.
    if (tid == 0) *s_abort = (int)ld_ag(a.abortw);
    __syncthreads();
    if (uni(*s_abort)) return;

    for (;;) {
        // ---- next system
        int sys = 0, n = h.n, R = h.R, K = Kg;
        int64_t r0 = 0;
        int c0 = 0;
        if constexpr (BATCH) {
            if (me == 0 && tid == 0) {
                // Own class first, then the classes of smaller gangs; none
                // once a gang has given up (the batch is repeated).
                int s = -1;
                for (int c = ld_ag(a.abortw) ? a.ncls : a.wg_class[blockIdx.x]; c < a.ncls && s < 0; ++c) {
                    const int q = a.cls_ptr[c] + atomicAdd(a.ticket + c, 1);
                    if (q < a.cls_ptr[c + 1]) s = a.order[q];
                }
                si[4] = s;
                if (Kg > 1) st_ag((int*)a.next_sys + first + turn, s);
            }
            GANG_ARRIVE();
            GANG_WAIT_FOR(Kg, epoch == 1 ? kWaitStart : kWaitSystem);
            if (Kg > 1 && tid == 0 && me != 0) si[4] = ld_ag((const int*)a.next_sys + first + turn);
            turn ^= 1;
            __syncthreads();
            sys = uni(si[4]);
            if (sys < 0) return;
            // A system is split over the gang size of its own class whichever
            // gang takes it, so its sums have one order and a repeated batch has
            // the same bits; a larger gang's other members wait.
            K = uni(a.sys_size[sys]);
            if (me >= K) {
                epoch += a.zcol_off[sys + 1] > a.zcol_off[sys] ? 2 : 1;   // the rendezvous of its start
                continue;
            }
            r0 = uni64(a.row_off[sys]);
            n = uni((int)(a.row_off[sys + 1] - r0));
            c0 = uni((int)a.zcol_off[sys]);
            R = uni((int)a.zcol_off[sys + 1] - c0);
        }
        const double* Einv = h.Einv + (BATCH ? uni64(a.e_off[sys]) : 0);
        const int RW = uni((((n + K - 1) / K) + 63) & ~63);   // positions per workgroup
        int nl = uni(h.vcap / (RW * (int)sizeof(VT)));            // basis columns in LDS
        nl = nl >= m ? kMP : (nl & ~7);
        const int p0 = me * RW;                            // first own position (system-local)
        VT* Vg = (VT*)h.V + (BATCH ? uni64(a.v_off[sys]) : 0);
        const int64_t ldv = BATCH ? (int64_t)((n + 1) & ~1) : h.ldv;
        WT* w = (WT*)h.w + (BATCH ? uni64(a.w_off[sys]) : 0);
        const BT* b = (const BT*)a.b + r0;
        double* x = a.xh + r0;
        const uint64_t t_start = wall_clock64();

        int pos[RPT];    // position in the workgroup (LDS index; 0 where there is none)
        int row[RPT];    // system-local row (0 where there is none)
        bool ok[RPT];
        bool wact = wv * kWave < RW;    // this wavefront holds rows
        // Its row slots in use (RW is a multiple of the wavefront): with three
        // or four slots a thread the basis loads of the others are skipped, and
        // in the dots those of rows that do not exist (the same solve: 31.4 ms
        // with a select per loaded entry instead, 26.7 so).
        const int qn = uni((RW - wv * kWave + kGN - 1) / kGN);
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            const int r = tid + q * kGN;
            ok[q] = r < RW && p0 + r < n;
            pos[q] = r < RW ? r : 0;
            row[q] = ok[q] ? (h.perm ? h.perm[p0 + r] : p0 + r) : 0;
        }
        // Basis storage, sums of idle wavefronts and coefficients start as
        // zero: rows past the end hold 0, slots past the last column repeat
        // it with coefficient 0.
        for (int i = tid; i < min(nl, m) * RW; i += kGN) Vl[i] = (ST)0;
        for (int i = tid; i < kGW * (kMP + 8 + kAU); i += kGN) red[0][i] = 0.0;
        // Place in global overflow columns (every row slot has a valid one): the
        // position, whose neighbours are the neighbouring lanes, unless the
        // basis is read by rows afterwards (265,225 sorted Q2 rows, FP32 basis:
        // 32.4 ms a mixed solve by rows, 31.4 by positions).
        int64_t gpos[RPT];
#pragma unroll
        for (int q = 0; q < RPT; ++q)
            gpos[q] = ADAPT ? (ok[q] ? row[q] : 0) : (ok[q] ? p0 + pos[q] : min(p0, n - 1));

        // Rows without A Z entries multiply s_0 by zero, listed or not.
        for (int i = tid; i < kMaxR; i += kGN) sv[i] = 0.0;
        // Own rows of the exchanges start empty.
        slot = pslot = pcount = tslot = 0;
        tpend = -1;
        if (K > 1)
            for (int i = tid; i < 3 * ps; i += kGN) st_empty(ring + ((i / ps) * K + me) * ps + i % ps);

        // ---- deflation lists of this workgroup
        int nz = 0, na = 0;
        if (R > 0) {
            if (tid < 32) bits[tid] = 0;
            __syncthreads();
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                if (ok[q]) {
                    const int64_t gi = r0 + row[q];
                    const int zc = a.zc1[gi];
                    if (zc >= 0) {
                        atomicOr(bits + ((zc - c0) >> 5), 1u << ((zc - c0) & 31));
                    } else if (zc == -2) {
                        for (int e = a.zrp[gi]; e < a.zrp[gi + 1]; ++e)
                            atomicOr(bits + ((a.zci[e] - c0) >> 5), 1u << ((a.zci[e] - c0) & 31));
                    }
                    const int a0 = a.az2c[2 * gi], a1 = a.az2c[2 * gi + 1];
                    if (a0 == -2) {
                        for (int e = a.azrp[gi]; e < a.azrp[gi + 1]; ++e)
                            atomicOr(bits + 8 + ((a.azci[e] - c0) >> 5), 1u << ((a.azci[e] - c0) & 31));
                    } else {
                        if (a0 >= 0) atomicOr(bits + 8 + ((a0 - c0) >> 5), 1u << ((a0 - c0) & 31));
                        if (a1 >= 0) atomicOr(bits + 8 + ((a1 - c0) >> 5), 1u << ((a1 - c0) & 31));
                    }
                }
            __syncthreads();
            if (tid < 8) {
                bits[8 + tid] |= bits[tid];   // the final correction needs s on Z's columns
                if (K > 1) st_ag(bmap + me * 8 + tid, bits[tid]);
            }
            __syncthreads();
            // Ordered lists: rank of a column = set bits below it.
            if (tid < R) {
                const int wd = tid >> 5;
                const unsigned below = (1u << (tid & 31)) - 1u;
                int rz = 0, ra = 0;
                for (int i = 0; i < wd; ++i) {
                    rz += __popc(bits[i]);
                    ra += __popc(bits[8 + i]);
                }
                if (bits[wd] >> (tid & 31) & 1u) zl[rz + __popc(bits[wd] & below)] = tid;
                if (bits[8 + wd] >> (tid & 31) & 1u) al[ra + __popc(bits[8 + wd] & below)] = tid;
                if (K > 1) {
                    // Entries of columns without own rows stay 0.
                    const bool own = (bits[wd] >> (tid & 31) & 1u) != 0;
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        if (own) st_empty(trow + (t * K + me) * ts + tid);
                        else st_ag(trow + (t * K + me) * ts + tid, 0.0);
                    }
                }
            }
            if (tid == 0) {
                int z = 0, c = 0;
                for (int i = 0; i < 8; ++i) {
                    z += __popc(bits[i]);
                    c += __popc(bits[8 + i]);
                }
                si[1] = z;
                si[2] = c;
            }
            GANG_ARRIVE();
            GANG_WAIT();
            nz = uni(si[1]);
            na = uni(si[2]);
            // Members that touch column t: [lo, hi).
            if (tid < R) {
                int lo = 0, hi = 1;
                if (K > 1) {
                    lo = K;
                    hi = 0;
                    for (int i = 0; i < K; ++i)
                        if (ld_ag(bmap + i * 8 + (tid >> 5)) >> (tid & 31) & 1u) {
                            lo = min(lo, i);
                            hi = i + 1;
                        }
                    if (hi == 0) lo = 0;
                }
                rng[tid] = lo | (hi << 16);
            }
            __syncthreads();
        }
        // Per row: rank of its Z column in the list (nz: none) and value; its
        // two A Z entries.  Rows with more entries (multi) take the CSR copies.
        int zi[RPT], ai0[RPT], ai1[RPT];
        ACC zvr[RPT], av0[RPT], av1[RPT];
        bool multi = false;
#pragma unroll
        for (int q = 0; q < RPT; ++q) {
            zi[q] = -1;
            ai0[q] = ai1[q] = 0;
            zvr[q] = av0[q] = av1[q] = 0;
            if (R > 0 && ok[q]) {
                const int64_t gi = r0 + row[q];
                const int zc = a.zc1[gi];
                if (zc >= 0) {
                    const int cz = zc - c0, wd = cz >> 5;
                    int rk = __popc(bits[wd] & ((1u << (cz & 31)) - 1u));
                    for (int i = 0; i < wd; ++i) rk += __popc(bits[i]);
                    zi[q] = rk;
                    zvr[q] = (ACC)a.zv1[gi];
                } else if (zc == -2) {
                    multi = true;
                }
                const int a0 = a.az2c[2 * gi], a1 = a.az2c[2 * gi + 1];
                if (a0 == -2) {
                    multi = true;
                } else {
                    if (a0 >= 0) {
                        ai0[q] = a0 - c0;
                        av0[q] = (ACC)((const AT*)a.az2v)[2 * gi];
                    }
                    if (a1 >= 0) {
                        ai1[q] = a1 - c0;
                        av1[q] = (ACC)((const AT*)a.az2v)[2 * gi + 1];
                    }
                }
            }
        }
        if (tid == 0) si[5] = 0;
        __syncthreads();
        if (multi) si[5] = 1;
        __syncthreads();
        multi = uni(si[5]) != 0;
        // Columns of the t sums (a power of two) and lanes per listed column of s.
        int RP = 16, EG = kWave;
        while (RP < R) RP <<= 1;
        while (EG > 8 && EG * na > kGN) EG >>= 1;
        // The rows of E^{-1} that the listed columns need, in LDS where they fit.
        const bool elds = na * R * 8 <= h.ecap;
        if (elds)
            for (int i = tid; i < na * R; i += kGN) {
                const int l = i / R, q = i - l * R;
                El[i] = h.trans ? Einv[(int64_t)al[l] * R + q] : Einv[(int64_t)q * R + al[l]];
            }

        // ---- pieces of a step
        // u = A xin on the own rows (xin: shared vector).  WF > 0: rows of at
        // most WF entries, held in registers for the whole solve.
        constexpr bool kKeepA = WF > 0;
        int mc[kKeepA ? RPT : 1][kKeepA ? WF : 1];
        AT mv[kKeepA ? RPT : 1][kKeepA ? WF : 1];
        auto slice_of = [&](int q, int64_t& off, int& wid) {
            const int64_t gp = h.perm ? p0 + pos[q] : r0 + row[q];   // global position
            const int64_t sl = gp >> 6;
            if (h.wuni > 0) {
                off = sl * h.wuni * kWave + (gp & 63);
                wid = h.wuni;
            } else {
                const int o0 = h.sell_off[sl];
                off = o0 + (gp & 63);
                wid = (h.sell_off[sl + 1] - o0) / kWave;
                if (wid == 0) off = 0;   // a slice of empty rows has no entry of its own
            }
        };
        auto mload = [&]() {
            if constexpr (WF > 0) {
#pragma unroll
                for (int q = 0; q < RPT; ++q) {
                    int64_t off = 0;
                    int wid = 0;
                    if (ok[q]) slice_of(q, off, wid);
                    // Branch-free: loads past the width repeat the last entry
                    // (entry 0 for rows that do not exist and slices without
                    // entries), and stand for 0 times the row's own element.
#pragma unroll
                    for (int k = 0; k < WF; ++k) {
                        const int64_t e = off + (int64_t)max(min(k, wid - 1), 0) * kWave;
                        mc[q][k] = (int)h.sell_col[e];
                        mv[q][k] = ((const AT*)h.sell_val)[e];
                    }
#pragma unroll
                    for (int k = 0; k < WF; ++k) {
                        mc[q][k] = k < wid ? mc[q][k] : 0;
                        mv[q][k] = k < wid ? mv[q][k] : (AT)0;
                    }
                }
            }
        };
        auto spmv = [&](auto* xin, ACC (&u)[RPT]) {
#pragma unroll
            for (int q = 0; q < RPT; ++q) u[q] = 0;
            if (!wact) return;
            if constexpr (kKeepA) {
                ACC xv[RPT][WF];
#pragma unroll
                for (int q = 0; q < RPT; ++q)
#pragma unroll
                    for (int k = 0; k < WF; ++k) {
                        GM_DCHECK(row[q] + mc[q][k] >= 0 && row[q] + mc[q][k] < n, kDbgSellCol);
                        xv[q][k] = (ACC)ld_ag(xin + row[q] + mc[q][k]);
                    }
#pragma unroll
                for (int q = 0; q < RPT; ++q)
#pragma unroll
                    for (int k = 0; k < WF; ++k) u[q] += (ACC)mv[q][k] * xv[q][k];
            } else {
                // Chunks of eight entries, the next chunk's entries requested
                // before this chunk's gathers are consumed.
                constexpr int CH = 8;
#pragma unroll
                for (int q = 0; q < RPT; ++q) {
                    int64_t off = 0;
                    int wid = 0;
                    if (ok[q]) slice_of(q, off, wid);
                    int cc[CH];
                    AT vv[CH];
#pragma unroll
                    for (int k = 0; k < CH; ++k) {
                        const int64_t e = off + (int64_t)max(min(k, wid - 1), 0) * kWave;
                        cc[k] = h.sell_col[e];
                        vv[k] = ((const AT*)h.sell_val)[e];
                    }
                    for (int k0 = 0; k0 < wid; k0 += CH) {
                        ACC xv[CH];
                        AT vc[CH];
#pragma unroll
                        for (int k = 0; k < CH; ++k) {
                            const int c = ok[q] ? cc[k] : 0;
                            GM_DCHECK(row[q] + c >= 0 && row[q] + c < n, kDbgSellCol);
                            xv[k] = (ACC)ld_ag(xin + row[q] + c);
                            vc[k] = vv[k];
                        }
#pragma unroll
                        for (int k = 0; k < CH; ++k) {
                            const int64_t e = off + (int64_t)min(k0 + CH + k, wid - 1) * kWave;
                            cc[k] = h.sell_col[e];
                            vv[k] = ((const AT*)h.sell_val)[e];
                        }
#pragma unroll
                        for (int k = 0; k < CH; ++k) u[q] += k0 + k < wid ? (ACC)vc[k] * xv[k] : (ACC)0;
                    }
                    if (!ok[q]) u[q] = 0;
                }
            }
        };
        // Z^T u partials of the own rows: tpart (K > 1) or tv.  Its last reads
        // of zred are not followed by a barrier: one has to come before coarse,
        // whose waves write zred whenever the sums they wait for are there.
        auto zt_out = [&](const ACC (&u)[RPT]) {
            for (int z0 = 0; z0 < nz; z0 += kZS) {
                const int ze = min(nz, z0 + kZS);
                if (z0 > 0) __syncthreads();
                for (int c = z0; c < ze; c += 8) {
                    ACC acc[8];
                    bool hit = false;
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] = 0;
#pragma unroll
                    for (int q = 0; q < RPT; ++q) {
                        const int d = zi[q] - c;
                        const ACC t = zvr[q] * u[q];
                        hit |= d >= 0 && d < 8;
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc[e] += d == e ? t : (ACC)0;
                    }
                    if (multi) {
#pragma unroll
                        for (int q = 0; q < RPT; ++q)
                            if (ok[q] && zi[q] < 0) {
                                const int64_t gi = r0 + row[q];
                                for (int e = a.zrp[gi]; e < a.zrp[gi + 1]; ++e)
#pragma unroll
                                    for (int l = 0; l < 8; ++l)
                                        if (c + l < ze && a.zci[e] - c0 == zl[c + l]) {
                                            acc[l] += (ACC)a.zv[e] * u[q];
                                            hit = true;
                                        }
                            }
                    }
                    ACC z = 0;
                    if (__any(hit)) z = gsum8(acc, ln);
                    const int l = c - z0 + gsum8_col(ln);
                    if ((ln & 7) == 0) zred[wv][l] = (double)z;
                }
                __syncthreads();
                const int l = z0 + tid;
                if (l < ze) {
                    double t = zred[0][tid];
#pragma unroll
                    for (int q = 1; q < kGW; ++q) t += zred[q][tid];
                    if (K > 1) st_ag(trow + (tslot * K + me) * ts + zl[l], t);
                    else tv[zl[l]] = t;
                }
            }
        };
        // s = E^{-1} t for the listed columns (after the rendezvous).
        auto coarse = [&]() {
            if (K > 1) {
                // Thread = (column, member in turn): lanes on neighbouring
                // columns read neighbouring entries of a member's row.
                const int col = tid & (RP - 1), cc = min(col, R - 1), G = kGN / RP;
                const int lo = rng[cc] & 0xffff, hi = rng[cc] >> 16;
                double t = 0;
                for (int i = lo + tid / RP; i < hi; i += 8 * G) {
                    unsigned long long v[8];
                    long long t0 = 0;
                    for (;;) {
                        bool wait = false;
#pragma unroll
                        for (int q = 0; q < 8; ++q)
                            v[q] = ld_bits(trow + (tslot * K + min(i + q * G, hi - 1)) * ts + cc);
#pragma unroll
                        for (int q = 0; q < 8; ++q) wait |= v[q] == kEmpty;
                        if (!wait) break;
                        const long long now = wall_clock64();
                        if (t0 == 0) t0 = now;
                        if (gang_expired(now - t0, h, a, kWaitSum)) {
                            *s_abort = 1;
                            break;
                        }
                    }
#pragma unroll
                    for (int q = 0; q < 8; ++q) t += i + q * G < hi ? __longlong_as_double((long long)v[q]) : 0.0;
                }
                tpend = tslot;
                tslot ^= 1;
                if (RP == 16) t = swap_add<false>(t, t);
                if (RP <= 32) t = swap_add<true>(t, t);
                const int W = min(RP, kWave);
                double* zr = &zred[0][0];
                if (ln < W) zr[RP <= kWave ? wv * W + ln : tid] = t;
                __syncthreads();
                if (tid < R) {
                    const int rows = RP <= kWave ? kGW : G;
                    t = zr[tid];
                    for (int q = 1; q < rows; ++q) t += zr[q * RP + tid];
                    tv[tid] = t;
                }
            } else if (tid < R && !(bits[tid >> 5] >> (tid & 31) & 1u)) {
                tv[tid] = 0.0;
            }
            __syncthreads();
            // EG lanes per listed column; (E^{-1})_{i,q} at Einv[q R + i]
            // (transposed for the adjoint).
            const int e0 = tid & (EG - 1);
            for (int l = tid / EG; l < na; l += kGN / EG) {
                const int i = al[l];
                double s = 0;
                if (elds) {
                    for (int q = e0; q < R; q += EG) s += El[l * R + q] * tv[q];
                } else {
                    const int64_t sr = h.trans ? 1 : R;
                    const double* er = Einv + (h.trans ? (int64_t)i * R : (int64_t)i);
                    for (int q = e0; q < R; q += 8 * EG) {
                        double v[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = er[min(q + e * EG, R - 1) * sr];
#pragma unroll
                        for (int e = 0; e < 8; ++e) s += q + e * EG < R ? v[e] * tv[q + e * EG] : 0.0;
                    }
                }
                s = ggroup_sum(s, EG);
                if (e0 == 0) sv[i] = s;
            }
            __syncthreads();
        };
        // u -= (A Z) s on the own rows.
        auto deflate = [&](ACC (&u)[RPT]) {
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                u[q] -= ok[q] ? av0[q] * (ACC)sv[ai0[q]] + av1[q] * (ACC)sv[ai1[q]] : (ACC)0;
            if (multi) {
#pragma unroll
                for (int q = 0; q < RPT; ++q) {
                    const int64_t gi = r0 + row[q];
                    if (ok[q] && a.az2c[2 * gi] == -2)
                        for (int e = a.azrp[gi]; e < a.azrp[gi + 1]; ++e)
                            u[q] -= (ACC)((const AT*)a.azv)[e] * (ACC)sv[a.azci[e] - c0];
                }
            }
        };
        // Eight consecutive basis columns c .. c+7 of row slot q (columns
        // past nv - 1 repeat it).  A chunk is in LDS or in global memory as a
        // whole: nl is a multiple of eight or covers every column.  A row that
        // does not exist reads its neighbour's entry, which may not have been
        // written yet: zero with drop, else for the caller to discard.
        auto vload = [&](int c, int nv, int q, ACC (&v)[8], bool drop = false) {
            if (c < nl) {
                const GM_LDS ST* bp = Vl + pos[q];
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = (ACC)bp[min(c + e, nv - 1) * RW];
            } else {
                const GM_GLB ST* bp = (const GM_GLB ST*)(Vg + gpos[q]);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const ACC t = (ACC)bp[min(c + e, nv - 1) * ldv];
                    v[e] = !drop || ok[q] ? t : (ACC)0;
                }
            }
        };
        // With three rows a thread their loads are kept apart: all in flight at
        // once they would not fit the registers.
        auto row_fence = [&]() {
            if constexpr (RPT > 2) __builtin_amdgcn_sched_barrier(0);
        };
        auto vput = [&](int k, int q, ACC v) -> ACC {   // returns the stored value
            const ST t = (ST)v;
            if (ok[q]) {
                if (k < nl) Vl[k * RW + pos[q]] = t;
                else ((GM_GLB ST*)Vg)[k * ldv + gpos[q]] = t;
            }
            return ok[q] ? (ACC)t : (ACC)0;
        };
        // Adaptive deflation: columns of U in use; y += (A U) C U^T x.
        const int ru = ADAPT ? uni(a.ast->r) : 0;
        // su = C tu with tu = ds[at ..] (a barrier follows in the caller).
        auto ucoarse = [&](int at) {
            for (int i = tid >> 3; i < ru; i += kGN / 8) {
                double t = 0;
                for (int q = tid & 7; q < ru; q += 8) t += a.aC[i * a.ald + q] * ds[at + q];
                t = ggroup_sum(t, 8);
                if ((tid & 7) == 0) su[i] = t;
            }
            __syncthreads();
        };
        auto ucorrect = [&](ACC (&u)[RPT]) {
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                if (!ok[q]) continue;
                const double* p = a.aAU + row[q];
                for (int c = 0; c < ru; c += 8) {
                    double v[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) v[e] = p[min(c + e, ru - 1) * h.ldv];
#pragma unroll
                    for (int e = 0; e < 8; ++e) u[q] += c + e < ru ? (ACC)(v[e] * su[c + e]) : (ACC)0;
                }
            }
        };
        // Publishes the own rows' partial dots of u with columns 0 .. nv-1 and
        // ||u||^2 (entry nv) and, with the adaptive deflation (ud), with the
        // columns of U (entries from nv + 1); with K = 1 they go to ds.
        auto dots = [&](int nv, const ACC (&u)[RPT], bool ud = false) {
            if (wact) {
                int c = 0;
                for (; c + 8 < nv; c += 16) {
                    ACC acc[16];
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[e] = 0;
#pragma unroll
                    for (int q = 0; q < RPT; ++q) {
                        if (RPT > 2 && !ok[q]) continue;
                        ACC v[8], v2[8];
                        vload(c, nv, q, v, RPT <= 2);
                        vload(c + 8, nv, q, v2, RPT <= 2);
#pragma unroll
                        for (int e = 0; e < 8; ++e) {
                            acc[e] += v[e] * u[q];
                            acc[8 + e] += v2[e] * u[q];
                        }
                        row_fence();
                    }
                    const ACC z = gsum16(acc, ln);
                    if ((ln & 3) == 0) red[wv][c + gsum16_col(ln)] = (double)z;
                }
                if (c < nv) {
                    ACC acc[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc[e] = 0;
#pragma unroll
                    for (int q = 0; q < RPT; ++q) {
                        if (RPT > 2 && !ok[q]) continue;
                        ACC v[8];
                        vload(c, nv, q, v, RPT <= 2);
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc[e] += v[e] * u[q];
                    }
                    const ACC z = gsum8(acc, ln);
                    if ((ln & 7) == 0) red[wv][c + gsum8_col(ln)] = (double)z;
                }
                if (ADAPT && ud)
                    for (int k = 0; k < ru; k += 8) {
                        ACC acc[8];
#pragma unroll
                        for (int e = 0; e < 8; ++e) acc[e] = 0;
#pragma unroll
                        for (int q = 0; q < RPT; ++q) {
                            const double* p = a.aU + row[q];
#pragma unroll
                            for (int e = 0; e < 8; ++e) acc[e] += (ACC)p[min(k + e, ru - 1) * h.ldv] * u[q];
                        }
                        const ACC z = gsum8(acc, ln);
                        if ((ln & 7) == 0) red[wv][kMP + 8 + k + gsum8_col(ln)] = (double)z;
                    }
                ACC t = 0;
#pragma unroll
                for (int q = 0; q < RPT; ++q) t += u[q] * u[q];
                t = gwave_sum(t);
                if (ln == 0) red[wv][kMP] = (double)t;
            }
            // Earlier stores (shared vectors, emptied rows) are in memory
            // before the row is published.
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (tid <= nv + (ADAPT && ud ? ru : 0)) {
                const int c = tid < nv ? tid : (tid == nv ? kMP : kMP + 8 + (tid - nv - 1));
                double t = red[0][c];
#pragma unroll
                for (int q = 1; q < kGW; ++q) t += red[q][c];
                if (K > 1) st_ag(ring + (slot * K + me) * ps + tid, t);
                else ds[tid] = t;
            }
        };
        // ds[0 .. nc-1] = the gang's sums of the published rows; false after
        // a timeout.
        auto collect = [&](int nc) -> bool {
            if (K > 1) {
                const double* part = ring + slot * K * ps;
                for (int c = 0; c < nc; c += kWave) {
                    const int left = nc - c;
                    if (left > 32) gang_rows<64>(left, part + c, ps, K, wv, ln, grow[wv] + c, s_abort, h, a);
                    else if (left > 16) gang_rows<32>(left, part + c, ps, K, wv, ln, grow[wv] + c, s_abort, h, a);
                    else gang_rows<16>(left, part + c, ps, K, wv, ln, grow[wv] + c, s_abort, h, a);
                }
                __syncthreads();
                if (tid < nc) {
                    double t = grow[0][tid];
#pragma unroll
                    for (int q = 1; q < kGW; ++q) t += grow[q][tid];
                    ds[tid] = t;
                }
                if (tid < pcount) st_empty(ring + (pslot * K + me) * ps + tid);
                if (tpend >= 0)
                    for (int l = tid; l < nz; l += kGN) st_empty(trow + (tpend * K + me) * ts + zl[l]);
                tpend = -1;
                pslot = slot;
                pcount = nc;
                slot = slot == 2 ? 0 : slot + 1;
            }
            __syncthreads();
            return !uni(*s_abort);
        };
#define COLLECT(nc)                        \
    do {                                   \
        if (!collect(nc)) GANG_FAIL();     \
    } while (0)

        // ---- start: r = b - A x
        int64_t its = a.resume ? uni64(a.ctrl->its) : 0;
        int cycles = a.resume ? uni(a.ctrl->cycles) : 0;
        int est_conv = a.resume ? uni(a.ctrl->est_conv) : 0;
        double rho0 = a.resume ? a.ctrl->rho0 : 0.0, target = a.resume ? a.ctrl->target : 0.0;
        int left = (int)min((int64_t)0x3fffffff, uni64(a.max_iters) - its);   // steps still allowed
        int status = kStatusOk, done = 0, bd = 0, kk = 0;
        double beta = 0.0;
        bool init = !a.resume;
        int launched = 0;
        mload();
        if (BATCH)   // batched: x starts from x0
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                if (ok[q]) st_ag(x + row[q], a.x0 ? a.x0[r0 + row[q]] : 0.0);
        GANG_ARRIVE();
        GANG_WAIT();
        bool fresh = true;
        for (;;) {
            ACC u[RPT];
            if (!fresh) COLLECT(1);   // every part of the iterate is in memory
            fresh = false;
            spmv(x, u);
            ACC nr = 0;
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                u[q] = ok[q] ? (ACC)(WT)((ACC)b[row[q]] - u[q]) : (ACC)0;
                nr += u[q] * u[q];
            }
            if (R > 0) zt_out(u);
            if (init) {
                dots(0, u);
                COLLECT(1);
                const double acc = unid(ds[0]);
                rho0 = a.r0_override > 0.0 ? a.r0_override : sqrt(acc);
                target = a.rtol * rho0;
                if (unib(!isfinite(acc) || !isfinite(rho0))) {
                    done = 1;
                    status = kStatusNonFinite;
                } else if (unib(rho0 == 0.0)) {
                    done = 1;
                }
                init = false;
            } else {
                __syncthreads();   // zt_out, then coarse
            }
            if (R > 0) {
                coarse();
                deflate(u);
            }
#pragma unroll
            for (int q = 0; q < RPT; ++q) u[q] = (ACC)(WT)u[q];
            if (done) break;
            dots(0, u);
            COLLECT(1);
            beta = sqrt(unid(ds[0]));
            if (unib(!isfinite(beta))) {
                done = 1;
                status = kStatusNonFinite;
            } else if (unib(beta <= target) || (a.trust_est && est_conv)) {
                done = 1;
            } else if (left <= 0) {
                done = 1;
                status = kStatusMaxIter;
            }
            if (done || launched >= a.max_cycles) break;
            ++launched;
            ++cycles;
            for (int i = tid; i < kMP; i += kGN) {
                c1[i] = 0;
                c2[i] = 0;
            }
            const double nscale = kHalf ? a.nscale : 1.0;
            const double vs = kHalf ? 1.0 / nscale : 1.0;      // stored -> normalised
            const ACC st0 = (ACC)(nscale / beta);
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                const ACC v = vput(0, q, u[q] * st0);
                if (ok[q]) st_ag(w + row[q], (WT)(v * (ACC)vs));
                u[q] = ADAPT ? v : (ACC)0;
            }
            if (tid == 0) gl[0] = beta;
            ACC wr[RPT];      // this thread's entries of the current vector
            dots(0, u, ADAPT);   // v_0 is in memory (the norm itself is not used)
            int j = 0;
            double wpre2 = 0.0;
            for (;; ++j) {
                // Step j: SpMV on w; meanwhile column j - 1 is finished.
                const bool last = j == m || (j > 0 && left <= 1);
                COLLECT((j > 0 ? j + 1 : 1) + (ADAPT ? ru : 0));
                if (!last) {
                    if (ADAPT && ru > 0) ucoarse(j > 0 ? j + 1 : 1);
                    spmv(w, u);
                    if (ADAPT && ru > 0) ucorrect(u);
#pragma unroll
                    for (int q = 0; q < RPT; ++q) u[q] = (ACC)(WT)u[q];
                    if (R > 0) {
                        zt_out(u);
                    }
                }
                double ihn = 0.0;   // 1 / hn of column j - 1
                if (j > 0) {
                    const int jc = j - 1;
                    double* hc = Hr + jc * (jc + 3) / 2;
                    // Every wave forms hn for itself; c = Hbar h2 (rows l <=
                    // jc; column jc is h1 + h2), eight lanes per row.
                    double q2 = 0;
                    for (int i = ln; i <= jc; i += kWave) {
                        const double v = ds[i] * vs;
                        q2 += v * v;
                        if (wv == 0) {
                            h2[i] = v;
                            hc[i] = h1[i] + v;
                        }
                    }
                    const double hn = sqrt(fmax(ds[j] - gwave_sum(q2), 0.0));
                    bd = unib(!(hn > 1.4901161193847656e-08 * sqrt(wpre2)));
                    ihn = bd ? 0.0 : 1.0 / hn;
                    const double h2l = ds[jc] * vs;
                    for (int l = tid >> 3; l <= jc; l += kGN / 8) {
                        double c = 0;
                        for (int k = (l > 0 ? l - 1 : 0) + (tid & 7); k < jc; k += 8)
                            c += Hr[k * (k + 3) / 2 + l] * (ds[k] * vs);
                        c = ggroup_sum(c, 8);
                        if ((tid & 7) == 0) {
                            const double hl = ds[l] * vs;
                            c += (h1[l] + hl) * h2l;
                            c2[l] = (ACC)(c * vs);
                            c1[l] = (ACC)(hl * vs);
                        }
                    }
                    if (tid == 0) hc[j] = hn;
                    ++its;
                    --left;
                }
                __syncthreads();
                if (j > 0 && tid == kGN - kWave) {
                    // Rotations of column j - 1 by one lane of the last wave
                    // (the others go on; the next barrier joins them).
                    const int jc = j - 1;
                    const double* hc = Hr + jc * (jc + 3) / 2;
                    const double hn = hc[j];
                    double av = hc[0];
                    for (int i = 0; i < jc; ++i) av = -sn[i] * av + cs[i] * hc[i + 1];
                    double rho = hypot(av, hn), cj = av / rho, sj = hn / rho;
                    if (hn == 0.0) {
                        cj = 1.0;
                        sj = 0.0;
                    }
                    cs[jc] = cj;
                    sn[jc] = sj;
                    const double gj = gl[jc];
                    gl[j] = -sj * gj;
                    gl[jc] = cj * gj;
                    const double est = fabs(sj * gj);
                    si[3] = est <= target ? 1 : 0;
                    if (me == 0 && !BATCH && a.hist) {
                        const int64_t hi = a.hist_base + its - 1;
                        if (hi < a.hist_cap) a.hist[hi] = est;
                    }
                }
                kk = j;
                if (last) break;
                if (R > 0) {
                    coarse();
                    deflate(u);
                }
                // Sweep A: the previous vector's second projection, v_j, the
                // new vector w_j = P A v_j (Arnoldi relation).
                if (j == 0) {
#pragma unroll
                    for (int q = 0; q < RPT; ++q) wr[q] = (ACC)(WT)u[q];
                } else {
                    const ACC ih = (ACC)ihn;
                    const ACC h2l = (ACC)h2[j - 1];
                    const ACC sg = kHalf ? (ACC)(ihn * nscale) : ih;
                    ACC a2[RPT], a3[RPT];
#pragma unroll
                    for (int q = 0; q < RPT; ++q) a2[q] = a3[q] = 0;
                    if (wact)
                        for (int c = 0; c < j; c += 8) {
                            ACC k2[8], k3[8];
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
                                k2[e] = c1[c + e];
                                k3[e] = c2[c + e];
                            }
#pragma unroll
                            for (int q = 0; q < RPT; ++q) {
                                if (RPT > 2 && q >= qn) continue;
                                ACC v[8];
                                vload(c, j, q, v);
#pragma unroll
                                for (int e = 0; e < 8; ++e) {
                                    a2[q] += v[e] * k2[e];
                                    a3[q] += v[e] * k3[e];
                                }
                                row_fence();
                            }
                        }
#pragma unroll
                    for (int q = 0; q < RPT; ++q) {
                        const ACC w2 = wr[q] - a2[q];
                        vput(j, q, ok[q] ? w2 * sg : (ACC)0);
                        wr[q] = ok[q] ? (ACC)(WT)((u[q] - a3[q] - w2 * h2l) * ih) : (ACC)0;
                    }
                }
                dots(j + 1, wr);
                COLLECT(j + 2);
                if (j > 0) {
                    // Column j - 1 ended the cycle (this step's sweep is dropped).
                    const int est = uni(si[3]);
                    if (est) est_conv = 1;
                    if (est || bd) break;
                }
                wpre2 = unid(ds[j + 1]);
                for (int i = tid; i <= j; i += kGN) {
                    const double h = ds[i] * vs;
                    h1[i] = h;
                    c1[i] = (ACC)(h * vs);
                }
                __syncthreads();
                // Sweep B: w -= V h1; the next SpMV's input.
                {
                    ACC a1[RPT];
#pragma unroll
                    for (int q = 0; q < RPT; ++q) a1[q] = 0;
                    if (wact)
                        for (int c = 0; c <= j; c += 8) {
                            ACC k1[8];
#pragma unroll
                            for (int e = 0; e < 8; ++e) k1[e] = c1[c + e];
#pragma unroll
                            for (int q = 0; q < RPT; ++q) {
                                if (RPT > 2 && q >= qn) continue;
                                ACC v[8];
                                vload(c, j + 1, q, v);
#pragma unroll
                                for (int e = 0; e < 8; ++e) a1[q] += v[e] * k1[e];
                                row_fence();
                            }
                        }
#pragma unroll
                    for (int q = 0; q < RPT; ++q) {
                        wr[q] = ok[q] ? (ACC)(WT)(wr[q] - a1[q]) : (ACC)0;
                        if (ok[q]) st_ag(w + row[q], (WT)wr[q]);
                    }
                }
                dots(j + 1, wr, ADAPT);
            }
            // After the last column: its estimate.
            __syncthreads();
            if (uni(si[3])) est_conv = 1;
            if (ADAPT && me == 0) {
                // The Ritz step outside reads the unrotated matrix.
                for (int i = tid; i < kk * (kk + 1); i += kGN) {
                    const int r = i / kk, q = i - r * kk;
                    if (r <= q + 1) a.Hraw[(int64_t)r * m + q] = Hr[q * (q + 3) / 2 + r];
                }
                __syncthreads();
            }
            // R from the unrotated columns (thread per column, in place), then
            // the back substitution by one wavefront (g and y in registers).
            __syncthreads();
            if (tid < kk) {
                double* hc = Hr + tid * (tid + 3) / 2;
                double av = hc[0];
                for (int i = 0; i < tid; ++i) {
                    const double bb = hc[i + 1];
                    hc[i] = cs[i] * av + sn[i] * bb;
                    av = -sn[i] * av + cs[i] * bb;
                }
                const double hn = hc[tid + 1];
                hc[tid] = hn == 0.0 ? av : hypot(av, hn);
            }
            __syncthreads();
            if (wv == 0) {
                double g0 = ln < kk ? gl[ln] : 0.0, g1 = ln + kWave < kk ? gl[ln + kWave] : 0.0;
                for (int i = kk - 1; i >= 0; --i) {
                    const double* hc = Hr + i * (i + 3) / 2;
                    const double gi = i < kWave ? __shfl(g0, i, kWave) : __shfl(g1, i - kWave, kWave);
                    const double yi = gi / hc[i];
                    if (ln < i) g0 -= hc[ln] * yi;
                    if (ln + kWave < i) g1 -= hc[ln + kWave] * yi;
                    if (ln == 0) ds[i] = yi * vs;
                }
            }
            __syncthreads();
            if constexpr (ADAPT) {
                // x += M^{-1} V y and the new Ritz vector are formed outside:
                // the basis goes to memory, its coefficients beside it.
#pragma unroll
                for (int q = 0; q < RPT; ++q)
                    if (ok[q])
                        for (int k = 0; k < min(kk, nl); ++k)
                            ((GM_GLB ST*)Vg)[k * ldv + gpos[q]] = Vl[k * RW + pos[q]];
                if (me == 0) {
                    if (tid < kk) a.coef[tid] = ds[tid];
                    if (tid <= kk) a.vscale[tid] = 1.0;
                    if (tid == 0 && a.cyc_k && cycles - 1 < a.cyc_cap) a.cyc_k[cycles - 1] = kk;
                }
                break;
            }
#pragma unroll
            for (int q = 0; q < RPT; ++q) {
                if (!ok[q]) continue;
                double acc = 0;
                for (int c = 0; c < kk; c += 8) {
                    ACC v[8];
                    vload(c, kk, q, v);
#pragma unroll
                    for (int e = 0; e < 8; ++e) acc += c + e < kk ? (double)v[e] * ds[c + e] : 0.0;
                }
                st_ag(x + row[q], ld_ag(x + row[q]) + acc);
            }
            if (me == 0 && tid == 0 && a.cyc_k && cycles - 1 < a.cyc_cap) a.cyc_k[cycles - 1] = kk;
#pragma unroll
            for (int q = 0; q < RPT; ++q) u[q] = 0;
            dots(0, u);
        }
        // ---- end of the solve (or of this launch's cycles)
        if (done || BATCH) {
            // x = x_hat + Z E^{-1} Z^T (b - A x_hat)
            double* xo = BATCH ? x : a.xout;
#pragma unroll
            for (int q = 0; q < RPT; ++q)
                if (ok[q]) {
                    const int64_t gi = r0 + row[q];
                    double v = ld_ag(x + row[q]);
                    if (R > 0 && rho0 > 0.0)
                        for (int e = a.zrp[gi]; e < a.zrp[gi + 1]; ++e) v += a.zv[e] * sv[a.zci[e] - c0];
                    xo[row[q]] = v;
                }
        }
        if (me == 0 && tid == 0) {
            if (BATCH) {
                a.out_i[3 * sys + 0] = its;
                a.out_i[3 * sys + 1] = cycles;
                a.out_i[3 * sys + 2] = status;
                a.out_d[4 * sys + 0] = rho0;
                a.out_d[4 * sys + 1] = rho0 > 0.0 ? beta / rho0 : 0.0;
                a.out_d[4 * sys + 2] = (double)t_start;
                a.out_d[4 * sys + 3] = (double)wall_clock64();
            } else {
                Ctrl* c = a.ctrl;
                c->its = its;
                c->cycles = cycles;
                c->done = done;
                c->stop = 1;
                c->status = status;
                c->k = kk;
                c->breakdown = bd;
                c->rho0 = rho0;
                c->target = target;
                c->beta = beta;
                c->est_conv = est_conv;
            }
        }
        if (!BATCH) return;
    }
}

// Clears the rendezvous words of a launch and puts its arguments in memory.
__global__ void k_gang_clear(GangArgs a, GangArgs* dst, unsigned* flags, int nwg, int nticket) {
    for (int i = threadIdx.x; i < nwg; i += blockDim.x) flags[i * kFlagW] = 0;
    for (int i = threadIdx.x; i < nticket; i += blockDim.x) a.ticket[i] = 0;
    if (threadIdx.x == 0) {
        *a.abortw = 0;
        *dst = a;
    }
}

// ------------------------------------------------------------------------ host
// The kernel for rpt row slots a thread, or null where no rule launches it: a
// batch's gangs have rows for one slot, three is the most for FP64, four for
// the reduced precisions.
template <typename AT, typename VT, typename WT, typename BT, typename ACC, int MODE>
static const void* gang_fn(int rpt, bool w9) {
    if (rpt == 1)
        return w9 ? (const void*)k_gang<AT, VT, WT, BT, ACC, 1, 9, MODE>
                  : (const void*)k_gang<AT, VT, WT, BT, ACC, 1, 0, MODE>;
    if constexpr (MODE != kGangBatch) {
        if (rpt == 2)
            return w9 ? (const void*)k_gang<AT, VT, WT, BT, ACC, 2, 9, MODE>
                      : (const void*)k_gang<AT, VT, WT, BT, ACC, 2, 0, MODE>;
        // No registers left for the matrix.
        if (rpt == 3) return (const void*)k_gang<AT, VT, WT, BT, ACC, 3, 0, MODE>;
        if constexpr (sizeof(VT) < 8)
            if (rpt == 4) return (const void*)k_gang<AT, VT, WT, BT, ACC, 4, 0, MODE>;
    }
    return nullptr;
}

size_t gang_lds_fixed(int m, int prec) {
    const size_t acc = prec == kPrecF64 ? 8 : 4;
    return 8 * (6 * (size_t)kMP + 2 * kAU + kGW * (kMP + 8 + kAU) + kGW * 2 * kWave + kGW * kZS + 2 * kMaxR) +
           2 * acc * kMP +
           4 * (3 * kMaxR + 32 + 8) + 256 + 8 * (size_t)gang_hraw(m);
}

size_t gang_args_bytes() { return sizeof(GangArgs); }

// Compute units of every die that the process's gangs hold, per device.
namespace {
struct Chip {
    std::mutex mu;
    std::condition_variable cv;
    int used = 0;
};
Chip g_chip[64];
}  // namespace

bool GangPlace::take(int device, int cus, int nwg, double wait_us) {
    if (device < 0 || device >= 64 || units_ > 0) return false;
    // Workgroups go round the dies, so a die gets at most one more than another.
    const int cap = std::max(1, cus / kXcd), need = std::min((nwg + kXcd - 1) / kXcd, cap);
    Chip& c = g_chip[device];
    std::unique_lock<std::mutex> lk(c.mu);
    if (!c.cv.wait_for(lk, std::chrono::duration<double, std::micro>(wait_us), [&] { return c.used + need <= cap; }))
        return false;
    c.used += need;
    device_ = device;
    units_ = need;
    return true;
}

GangPlace::~GangPlace() {
    if (units_ == 0) return;
    Chip& c = g_chip[device_];
    {
        std::lock_guard<std::mutex> lk(c.mu);
        c.used -= units_;
    }
    c.cv.notify_all();
}

bool launch_gang(const GangHot& h0, const GangArgs& a, void* args_d, int prec, int rpt, bool w9, int nwg,
                 int nticket) {
    GangHot h = h0;
    const void* f = a.row_off          ? gang_fn<double, double, double, double, double, kGangBatch>(rpt, w9)
                    : a.ast            ? gang_fn<double, double, double, double, double, kGangAdapt>(rpt, w9)
                    : prec == kPrecF64 ? gang_fn<double, double, double, double, double, kGangSingle>(rpt, w9)
                    : prec == kPrecF32 ? gang_fn<float, float, float, float, float, kGangSingle>(rpt, w9)
                                       : gang_fn<float, __half, float, float, float, kGangSingle>(rpt, w9);
    if (!f) return false;
    const size_t dynb = 8 * (size_t)gang_hraw(h.m) + h.ecap + h.vcap;
    if (hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dynb) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    GangArgs* ad = static_cast<GangArgs*>(args_d);
    k_gang_clear<<<1, 256, 0, a.st>>>(a, ad, h.flags, nwg, nticket);
    const GangArgs* ac = ad;
    void* args[] = {&h, &ac};
    if (hipLaunchKernel(f, dim3(nwg), dim3(kGN), args, dynb, a.st) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return true;
}

GM_DEBUG_ACCESSOR(dbg_take_gang)

}  // namespace gm

// The diamond-difference transport sweep (paper section II.B, eqs. 8-22)
// for gfx950 (CDNA4, wave64): the kernel, its launch shapes and launcher.
// See internal.h for the pencil voxel layout.
#include <hip/hip_runtime.h>
#include <math.h>

#include <type_traits>

#include "internal.h"

namespace dsn {

template <typename T>
__device__ __forceinline__ T dd_div(T num, T den)
{
    return num / den;
}
template <>
__device__ __forceinline__ float dd_div<float>(float num, float den)
{
    return num * __builtin_amdgcn_rcpf(den);
}

// ---------------------------------------------------------------------------
// a2: diamond-difference transport sweep.
//
// One wave = one direction x one pencil (8 x 8 columns of voxels spanning the
// x extent).  Lane (j, k) marches along x with a diagonal skew: at step s it
// updates the voxel with i_r + j_r + k_r = s (octant-relative indices), i.e.
// each step is one sub-sweep plane (section II.B) restricted to the pencil.
// The x inflow stays in a register; y and z inflows are the neighbouring
// lanes' outflows of the previous step (cross-lane permute), or the upstream
// pencil's outgoing face on the pencil boundary.
//
// Memory: the skew makes one step touch 15 different 64-voxel rows, so Q/psi
// rows are staged through a per-wave LDS ring and every global access of
// Q/psi moves whole rows; the details are with k_sweep below.
// ---------------------------------------------------------------------------
// Cross-lane moves in the step phase.  There lane L stands for the
// octant-relative column (j_r, k_r) = (L & 7, L >> 3), so the upstream
// neighbours are always lanes L-1 (y) and L-8 (z) whatever the octant.  The y
// move is a whole-wave DPP shift; lanes with j_r = 0 (k_r = 0) take the face
// inflow instead, so the values shifted across column ends are never used.
__device__ __forceinline__ float lane_shr1(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x138, 0xF, 0xF, true));
}
__device__ __forceinline__ double lane_shr1(double v)
{
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)(x & 0xffffffffLL), 0x138, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(x >> 32), 0x138, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ float lane_from(float v, int src_byte)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(src_byte, __float_as_int(v)));
}
__device__ __forceinline__ double lane_from(double v, int src_byte)
{
    const long long x = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_ds_bpermute(src_byte, (int)(x & 0xffffffffLL));
    const int hi = __builtin_amdgcn_ds_bpermute(src_byte, (int)(x >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

__device__ __forceinline__ float fmin3(float a, float b, float c) { return fminf(fminf(a, b), c); }
__device__ __forceinline__ double fmin3(double a, double b, double c) { return fmin(fmin(a, b), c); }

// Cell modes of the sweep (the sweep_mode of the argument block):
//   kDD      pure diamond difference
//   kFixup   with the set-to-zero fixup
//   kRecord  with the fixup, and the set of fixed axes of every cell written
//            to mk (bit a: axis a fixed)
//   kTrans   the transpose of the fixup cell with the fixed set mk frozen,
//            for the adjoint sweep along -Omega: psi = (q + sum over free
//            axes of c_a in_a) / (sigma + sum over free axes of c_a), outflow
//            2 psi - in_a on a free axis and psi on a fixed one (reverse-mode
//            differentiation of the frozen cell, adjoint face values scaled
//            by 2 / c_a)
constexpr int kDD = 0, kFixup = 1, kRecord = 2, kTrans = 3;

// z_ready(oz) is called with every value of the z outflow, the last one final:
// the tile sweep starts its move to the neighbour lane there, before the fixup's
// test (the move is on the step's critical path, and the fixup is rare).
struct NoHook {
    template <typename T>
    __device__ void operator()(T) const
    {
    }
};
template <typename T, int MODE, typename Z = NoHook>
__device__ __forceinline__ T dd_update(T q, T sg, T cx, T cy, T cz, T csum, T px, T iny, T inz, T &ox_, T &oy_,
                                       T &oz_, unsigned &mk, Z z_ready = Z())
{
    if constexpr (MODE == kTrans) {
        const T kx = (mk & 1u) ? T(0) : T(1), ky = (mk & 2u) ? T(0) : T(1), kz = (mk & 4u) ? T(0) : T(1);
        const T p = dd_div<T>(q + kx * cx * px + ky * cy * iny + kz * cz * inz, sg + kx * cx + ky * cy + kz * cz);
        ox_ = (mk & 1u) ? p : T(2) * p - px;
        oy_ = (mk & 2u) ? p : T(2) * p - iny;
        oz_ = (mk & 4u) ? p : T(2) * p - inz;
        z_ready(oz_);
        return p;
    }
    const T num0 = q + cx * px + cy * iny + cz * inz, den0 = sg + csum;
    T p = dd_div<T>(num0, den0);
    ox_ = T(2) * p - px;
    oy_ = T(2) * p - iny;
    oz_ = T(2) * p - inz;
    z_ready(oz_);
    if constexpr (MODE == kFixup || MODE == kRecord) {
        // Set-to-zero fixup.  An axis whose outflow is negative is fixed
        // (m_a = 1): its outflow becomes zero, its inflow enters the balance
        // with half weight and its coefficient leaves the denominator; the
        // cell is re-solved, and axes that turn negative are fixed in the
        // next pass (at most three).  A pass in which no axis of a lane turns
        // negative reproduces that lane's values exactly, so the passes run
        // branch-free over the whole wave while any lane still needs one.
        T lo = fmin3(ox_, oy_, oz_);
        if (__any(lo < T(0))) {
            T mx = T(0), my = T(0), mz = T(0);
            const T hx = T(0.5) * cx * px, hy = T(0.5) * cy * iny, hz = T(0.5) * cz * inz;
#pragma unroll
            for (int pass = 0; pass < 3; ++pass) {
                mx = ox_ < T(0) ? T(1) : mx;
                my = oy_ < T(0) ? T(1) : my;
                mz = oz_ < T(0) ? T(1) : mz;
                const T num = num0 - (mx * hx + my * hy + mz * hz);
                const T den = den0 - (mx * cx + my * cy + mz * cz);
                p = dd_div<T>(num, den);
                ox_ = mx != T(0) ? T(0) : T(2) * p - px;
                oy_ = my != T(0) ? T(0) : T(2) * p - iny;
                oz_ = mz != T(0) ? T(0) : T(2) * p - inz;
                if (pass == 2) break;
                lo = fmin3(ox_, oy_, oz_);
                if (!__any(lo < T(0))) break;
            }
            if constexpr (MODE == kRecord)
                mk = (mx != T(0) ? 1u : 0u) | (my != T(0) ? 2u : 0u) | (mz != T(0) ? 4u : 0u);
            z_ready(oz_);
        }
    }
    return p;
}

// Values that no kernel writes while a sweep runs, read through the constant
// address space: uniform ones become scalar loads, which the waves of a CU
// share through the scalar cache.  As vector loads of a few shared lines by
// every wave of a launch they took 10 us to come back.
template <typename X>
__device__ __forceinline__ X const_load(const X *p)
{
    return *(const __attribute__((address_space(4))) X *)p;
}

// Device-coherent (agent scope) loads and stores: they bypass the per-XCD
// L2, so a block on any XCD sees them.
template <typename T>
__device__ __forceinline__ T coherent_load(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void coherent_store(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Buffer resources for the sweep's memory traffic.  Every load and store of
// the chunk loop is issued unconditionally: a row outside the pencil gets an
// offset beyond its buffer's size (a row before the first wraps to an
// unsigned offset of 2^31 or more; every buffer is below 2 GiB), so the
// hardware range check turns its load into zero and drops its store.  With
// no branches around memory instructions the compiler waits only for the
// loads it needs, never for the completion of earlier stores.
typedef __amdgpu_buffer_rsrc_t Rsrc;
typedef __attribute__((ext_vector_type(2))) unsigned U32x2;
typedef __attribute__((ext_vector_type(4))) unsigned U4;
constexpr int kDstLds = 256;            // diagonal-start table entries kept in LDS
constexpr int kSigTab = 32;             // per-block sigma table: materials < kMaxMat, the ghost byte 255 -> 31
static_assert(kMaxMat <= 16, "the ghost byte must land on a zero entry of the sigma table");
constexpr int kTicketStop = 1 << 30;     // ticket counter after an abort (above any item count)
constexpr int kRawDword3 = 0x00020000;   // raw (untyped) 32-bit buffer access
constexpr int kSC1 = 16;                 // device-coherent: bypasses the per-XCD L2
constexpr int kVolatileSC1 = (int)0x80000010u;
constexpr int kSC0 = 1;                  // bypasses the CU's L1, coherent in the XCD's L2
constexpr int kVolatileSC0 = (int)0x80000001u;
constexpr int kNT = 2;                   // non-temporal: streamed data, not kept in the caches

__device__ __forceinline__ Rsrc make_rsrc(const void *base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, kRawDword3);
}
// The same, for an address that is the same in every lane of a wave but that
// the compiler cannot prove to be (else it would loop over the lanes' values
// around every access).
__device__ __forceinline__ Rsrc make_uniform_rsrc(const void *base, unsigned bytes)
{
    const unsigned long long p = (unsigned long long)base;
    const unsigned lo = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)p);
    const unsigned hi = (unsigned)__builtin_amdgcn_readfirstlane((int)(unsigned)(p >> 32));
    return make_rsrc((const void *)((unsigned long long)hi << 32 | lo),
                     (unsigned)__builtin_amdgcn_readfirstlane((int)bytes));
}
template <int AUX = 0>
__device__ __forceinline__ float buf_load(Rsrc r, unsigned off, float)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, AUX));
}
template <int AUX = 0>
__device__ __forceinline__ double buf_load(Rsrc r, unsigned off, double)
{
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, AUX);
    return __longlong_as_double((long long)(((unsigned long long)v[1] << 32) | v[0]));
}
template <int AUX = 0>
__device__ __forceinline__ void buf_store(Rsrc r, unsigned off, float x)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(x), r, off, 0, AUX);
}
template <int AUX = 0>
__device__ __forceinline__ void buf_store(Rsrc r, unsigned off, double x)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    __builtin_amdgcn_raw_buffer_store_b64(U32x2{(unsigned)b, (unsigned)(b >> 32)}, r, off, 0, AUX);
}

// Face words.  An upstream block publishes face values that a downstream
// block polls; each word carries a stamp of the sweep that wrote it, in the
// same naturally aligned word as the data (single-copy atomic), so a reader
// that sees the current stamp has that word's data: no separate flag and no
// wait for store completion.  Stores and polls are device-coherent, except
// in the per-XCD-queue sweeps, where producer and consumer share one XCD and
// its L2 (plain stores, loads that bypass only the CU's L1).
//
// TaggedFace<T>: every 32-bit half of a value in one 64-bit word {half,
// epoch}; the epoch grows with every sweep launch.  Works for any value.
//
// SignFace<T>: for sweeps with the set-to-zero fixup, whose outflows are
// never negative, the value without its sign bit (one 32-bit word in FP32,
// one 64-bit word in FP64) and in the sign bit a per-source parity that
// flips after every sweep in which the source ran.
// A word left from that source's previous sweep has the other parity; words
// older than that never survive, because every sweep of a source rewrites all
// its face words.  All-ones (a NaN) is never accepted, which is how freshly
// allocated or invalidated faces read.
template <typename T>
struct TaggedFace {
    static constexpr int N = sizeof(T) / 4;  // 64-bit words per value
    static constexpr unsigned BYTES = 8 * N;
    typedef U32x2 Word[N];
    template <int AUX>
    static __device__ __forceinline__ void load(Word &w, Rsrc r, unsigned off)
    {
#pragma unroll
        for (int q = 0; q < N; ++q) w[q] = __builtin_amdgcn_raw_buffer_load_b64(r, off + 8 * q, 0, AUX);
    }
    static __device__ __forceinline__ bool ok(const Word &w, unsigned stamp)
    {
        bool good = true;
#pragma unroll
        for (int q = 0; q < N; ++q) good = good && w[q][1] == stamp;
        return good;
    }
    static __device__ __forceinline__ T value(const Word &w)
    {
        if constexpr (N == 1)
            return __uint_as_float(w[0][0]);
        else
            return __longlong_as_double((long long)(((unsigned long long)w[1][0] << 32) | w[0][0]));
    }
    template <int AUX>
    static __device__ __forceinline__ void put(Rsrc r, unsigned off, T v, unsigned stamp)
    {
        if constexpr (N == 1) {
            __builtin_amdgcn_raw_buffer_store_b64(U32x2{__float_as_uint(v), stamp}, r, off, 0, AUX);
        } else {
            const unsigned long long b = (unsigned long long)__double_as_longlong(v);
            __builtin_amdgcn_raw_buffer_store_b64(U32x2{(unsigned)b, stamp}, r, off, 0, AUX);
            __builtin_amdgcn_raw_buffer_store_b64(U32x2{(unsigned)(b >> 32), stamp}, r, off + 8, 0, AUX);
        }
    }
};
template <typename T>
struct SignFace;
template <>
struct SignFace<float> {
    static constexpr unsigned BYTES = 4;
    typedef unsigned Word;
    template <int AUX>
    static __device__ __forceinline__ void load(Word &w, Rsrc r, unsigned off)
    {
        w = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, AUX);
    }
    static __device__ __forceinline__ bool ok(Word w, unsigned parity)
    {
        return (w ^ (parity << 31)) <= 0x7F800000u;  // the parity bit matches and the rest is no NaN
    }
    static __device__ __forceinline__ float value(Word w) { return __uint_as_float(w & 0x7FFFFFFFu); }
    template <int AUX>
    static __device__ __forceinline__ void put(Rsrc r, unsigned off, float v, unsigned parity)
    {
        __builtin_amdgcn_raw_buffer_store_b32((__float_as_uint(v) & 0x7FFFFFFFu) | (parity << 31), r, off, 0, AUX);
    }
};
template <>
struct SignFace<double> {
    static constexpr unsigned BYTES = 8;
    typedef U32x2 Word;  // {low half, high half with the parity in bit 31}
    template <int AUX>
    static __device__ __forceinline__ void load(Word &w, Rsrc r, unsigned off)
    {
        w = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, AUX);
    }
    static __device__ __forceinline__ bool ok(const Word &w, unsigned parity)
    {
        const unsigned hi = w[1] & 0x7FFFFFFFu;
        return (w[1] >> 31) == parity && (hi < 0x7FF00000u || (hi == 0x7FF00000u && w[0] == 0u));
    }
    static __device__ __forceinline__ double value(const Word &w)
    {
        return __longlong_as_double((long long)(((unsigned long long)(w[1] & 0x7FFFFFFFu) << 32) | w[0]));
    }
    template <int AUX>
    static __device__ __forceinline__ void put(Rsrc r, unsigned off, double v, unsigned parity)
    {
        const unsigned long long b = (unsigned long long)__double_as_longlong(v);
        const unsigned hi = ((unsigned)(b >> 32) & 0x7FFFFFFFu) | (parity << 31);
        __builtin_amdgcn_raw_buffer_store_b64(U32x2{(unsigned)b, hi}, r, off, 0, AUX);
    }
};
// Fixup sweeps (outflows never negative) carry the sign-parity words; pure DD
// and transposed sweeps the tagged ones, and so do the per-XCD-queue sweeps:
// their face words live in an XCD's L2, and only an epoch that is new with
// every launch makes a line left there by an earlier launch unacceptable.
template <typename T, int MODE, bool XCD>
struct FaceCodecSel {
    typedef typename std::conditional<!XCD && (MODE == kFixup || MODE == kRecord), SignFace<T>, TaggedFace<T>>::type
        type;
};

// Material bytes of octant-relative rows 8c .. 8c+7 of a pencil (64 bytes
// per row, one per column): physically 512 contiguous bytes, which lane l
// loads 8 at a time (physical row l / 8 of the block, columns 8 (l mod 8)
// .. 8 (l mod 8) + 7).  Rows outside the pencil lie outside the buffer and
// read as zero; a lane's 8 bytes never straddle two rows.
__device__ __forceinline__ U32x2 load_mat_rows(Rsrc r, int c, int sx, int nx, int lane)
{
    const int row0 = sx > 0 ? 8 * c : nx - 8 - 8 * c;  // physical row at the start of the block
    const auto v = __builtin_amdgcn_raw_buffer_load_b64(r, (unsigned)(row0 * 64 + 8 * lane), 0, 0);
    return U32x2{v[0], v[1]};
}
// octant-relative row (within the chunk) of the bytes lane l loaded
__device__ __forceinline__ int mat_row(int sx, int lane) { return sx > 0 ? lane >> 3 : 7 - (lane >> 3); }

// sigma in the sweep.  SM = false: the group's sigma_t array (pencil order,
// type T).  SM = true (no per-voxel density, so sigma_t depends on the
// material only): one byte per voxel, the material, looked up in a per-block
// table of the group's cross sections (index 255, the ghost, maps to zero).
template <typename T, bool SM>
struct SigSrc;
template <typename T>
struct SigSrc<T, false> {
    typedef T Reg;
    static constexpr int ROW = 64 * sizeof(T);  // bytes per pencil row
    static __device__ __forceinline__ Reg load(Rsrc r, unsigned off) { return buf_load(r, off, T()); }
    static __device__ __forceinline__ T value(Reg x, const T *) { return x; }
};
template <typename T>
struct SigSrc<T, true> {
    typedef unsigned Reg;
    static constexpr int ROW = 64;
    static __device__ __forceinline__ Reg load(Rsrc r, unsigned off)
    {
        return __builtin_amdgcn_raw_buffer_load_b8(r, off, 0, 0);
    }
    static __device__ __forceinline__ T value(Reg x, const T *table) { return table[x]; }
};

// Persistent, pipelined sweep of all directions.
//
// Work item = (octant o, group of WPB directions dg, pencil (J_r, K_r),
// source), one block; wave w of the block sweeps direction dg * WPB + w.
// Blocks take tickets from a global counter; tickets are numbered by pencil
// diagonal J_r + K_r first, so an item's upstream pencils (J_r - 1, K_r) and
// (J_r, K_r - 1) always hold smaller tickets, i.e. they were taken by blocks
// that are already running: no block waits on work that has not started, and
// every wait ends.
//
// Pipelining: outgoing face rows are published as soon as each 8-step chunk
// completes them; a downstream wave reads the face rows of its next chunk
// ahead of time and, when it commits them, re-reads any word whose stamp is
// not yet the current sweep's.  Downstream pencils therefore run a couple of
// chunks behind their upstream neighbours instead of waiting for whole
// pencils (KBA-style pipelining inside one GPU).  Every wait is bounded; on
// timeout the wave raises a global abort flag, the block leaves at its next
// ticket, and the host reports an error.
//
// Per wave and chunk c (steps t = 8c .. 8c+7; lane (j_r, k_r) updates row
// i_r = t - j_r - k_r at step t):
//   - psi (holding the source Q on entry) rows 8c .. 8c+7 are loaded a chunk
//     ahead as whole rows and committed to an LDS ring (row r in slot
//     r mod 24); steps read and overwrite them in place; rows 8c-16 .. 8c-9
//     are complete and go back to memory as whole rows;
//   - with sigma from the material (SM), the material bytes of rows 8c ..
//     8c+7 ride with the psi rows: whole rows, loaded a chunk ahead, into a
//     byte ring in LDS with the same slots; each step reads the byte of the
//     lane's own cell and looks sigma up in the block's table.  With
//     sigma in memory (per-voxel density), each lane reads sigma of its own
//     column for the next chunk's rows straight from memory, one load per
//     step right after that step has used the current value;
//   - face rows are stored skewed: a face value of row r needed (or made)
//     by a lane with skew s at step r + s sits in ring slot (r + s) mod 16,
//     so every step reads and writes one slot common to all lanes.
// Waves of a block share nothing but the ticket, so there is no barrier
// inside an item.  In FP32 the register budget is held to four waves per
// SIMD (16 per CU, e.g. four blocks of four directions) where the LDS allows
// that many.
//
// XCD (sweep_xcd = nq > 0): octant o is swept only by blocks running on XCD
// o mod nq, which take tickets from that XCD's own counter; all pencils of a
// direction then run on one XCD, so the face words between them need only
// be coherent in that XCD's L2 (plain stores, loads that bypass only the
// CU's L1).  Each block takes its queue from the XCD it runs on
// (hardware register XCC_ID), so a queue's blocks always share one L2.  The
// runtime enables it only after seeing consecutive workgroups go to
// consecutive XCDs (round robin; the first XCD depends on the hardware
// queue) and launches a whole number of blocks per XCD; a check after the
// launch reports any queue that no block served.
//
// NT: the psi rows are loaded and stored non-temporally (the runtime sets it
// when the launch's angular fluence exceeds the last-level cache, so that
// the streamed rows do not displace the face words and material bytes).
//
// MULTI: several problems (meshes) in one launch (k_sweep_multi): a0.multi
// holds their argument blocks and a0.seg the merged ticket order; an item's
// geometry, arrays and cross sections are its own problem's.
template <typename T, int MODE, int WPB, bool SM, bool XCD, bool NT, bool MULTI>
__device__ __forceinline__ void sweep_body(const SolveArgs<T> &a0, int g)
{
    constexpr int kLoadAux = XCD ? kSC0 : kSC1, kPollAux = XCD ? kVolatileSC0 : kVolatileSC1;
    constexpr int kStoreAux = XCD ? 0 : kSC1;
    constexpr int kPsiAux = NT ? kNT : 0;
    typedef SigSrc<T, SM> Sig;
    typedef typename FaceCodecSel<T, MODE, XCD>::type Face;
    constexpr bool kSignFace = std::is_same<Face, SignFace<T>>::value;
    constexpr int RQ = 24, RF = 16, CH = 8;
    constexpr int RB = 64 * sizeof(T);          // bytes per pencil row
    constexpr int FB = 8 * (int)Face::BYTES;    // bytes per face row
    __shared__ T sQ[WPB][RQ][64];
    __shared__ T sFYi[WPB][RF][8], sFZi[WPB][RF][8], sFYo[WPB][RF][8], sFZo[WPB][RF][8];
    __shared__ int sTicket;
    __shared__ int sDst[kDstLds];  // first ticket of every pencil diagonal, when it fits
    __shared__ T sSigT[SM ? kSigTab : 1];
    __shared__ __align__(16) unsigned char sMt[SM ? WPB : 1][SM ? RQ : 1][64];  // SM: material byte ring (slots as sQ)
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int D = a0.D, ngrp = D / WPB;
    constexpr bool multi = MULTI;
    // [0] next ticket (an abort lifts it to kTicketStop, so every later ticket
    // is past the end), [1] abort flag for the host, [2] epoch, [kQueueCtr +
    // q] next ticket of XCD q's queue
    int *const ctr = a0.sweep_ctr;
    const unsigned epoch = (unsigned)ctr[2];  // set after the sweep before this one
    const int nq = XCD ? a0.sweep_xcd : 1;
    const int xq = XCD ? (int)__builtin_amdgcn_readfirstlane(__builtin_amdgcn_s_getreg((3 << 11) | 20)) % nq : 0;
    int *const tctr = XCD ? &ctr[kQueueCtr + xq] : &ctr[0];  // this block's ticket counter
    const int nitems = XCD ? a0.sweep_nitems / nq : a0.sweep_nitems;

    // An iteration enqueued after every source's group converged does
    // nothing: leave before touching the ticket queue.
    bool live = false;
    if constexpr (MULTI) {
        for (int q = 0; q < a0.nmulti; ++q) {
            const SolveArgs<T> &aq = a0.multi[q];
            for (int s = 0; s < aq.S; ++s) live = live || !aq.ctl[(long)s * aq.G + g].done;
        }
    } else {
        for (int s = 0; s < a0.S; ++s) live = live || !a0.ctl[(long)s * a0.G + g].done;
    }
    if (!live) return;
    int sig_of = -1;  // problem whose cross sections sSigT holds
    if (SM && !multi) {
        for (int i = threadIdx.x; i < kSigTab; i += 64 * WPB)
            sSigT[i] = i < a0.nmat ? (T)a0.xs_t[i * a0.G + g] : T(0);
        sig_of = 0;
    }
    // first ticket of every pencil diagonal (of every segment when multi)
    const int ndiag = multi ? a0.nseg : a0.g.NJ + a0.g.NK - 1;
    const int *const dstart = multi ? a0.seg : a0.sweep_dstart;
    const bool dst_lds = ndiag <= kDstLds;
    if (dst_lds)
        for (int i = threadIdx.x; i < ndiag; i += 64 * WPB) sDst[i] = dstart[i];
    // The next item's ticket is taken three chunks before an item ends, so
    // the atomic's latency hides behind those chunks while a ticket held in
    // advance (possibly the upstream of another block's item) waits at most
    // three chunks.  A block holds at most two tickets, the one it works on
    // and the next; the smallest unfinished ticket is therefore always being
    // worked on, and its upstream items (smaller tickets) are finished: the
    // queue always makes progress.
    int tnext = 0;
    bool have_next = false;  // thread 0 only
    for (;;) {
        if (threadIdx.x == 0) {
            sTicket = have_next ? tnext : atomicAdd(tctr, 1);
            have_next = false;
        }
        __syncthreads();
        const int t = __builtin_amdgcn_readfirstlane(sTicket);
        __syncthreads();
        if (t >= nitems) break;
        const int tq = t * nq;  // an XCD queue's diagonal starts are the global ones / nq
        // ticket -> (diagonal, position, direction group, octant, source); the
        // diagonal starts increase, so d = #{starts of diagonals 1.. <= t}
        int d = 0;
        if (dst_lds) {
            for (int base = 1; base < ndiag; base += 64) {
                const int i = base + lane;
                d += __popcll(__ballot(i < ndiag && sDst[i] <= tq));
            }
            d = __builtin_amdgcn_readfirstlane(d);
        } else {
            // the largest d with dstart[d] <= tq (starts strictly increase)
            int hi = ndiag - 1;
            while (d < hi) {
                const int mid = (d + hi + 1) >> 1;
                if (dstart[mid] <= tq) d = mid;
                else hi = mid - 1;
            }
        }
        int u = t - (dst_lds ? __builtin_amdgcn_readfirstlane(sDst[d]) : dstart[d]) / nq;
        // the item's problem and its pencil diagonal
        int pi = 0;
        if constexpr (MULTI) {
            const int code = a0.seg[ndiag + 1 + d];
            pi = code >> 16;
            d = code & 0xFFFF;
        }
        const SolveArgs<T> &A = MULTI ? a0.multi[pi] : a0;
        if (SM && pi != sig_of) {  // uniform over the block; no wave is inside an item
            for (int i = threadIdx.x; i < kSigTab; i += 64 * WPB)
                sSigT[i] = i < A.nmat ? (T)A.xs_t[i * A.G + g] : T(0);
            __syncthreads();
            sig_of = pi;
        }
        const int NJ = A.g.NJ, NK = A.g.NK, nx = A.g.nx;
        const long Vp = A.g.Vp;
        const int Jlo = d - (NK - 1) > 0 ? d - (NK - 1) : 0;
        const int Jhi = d < NJ - 1 ? d : NJ - 1;
        const int P = Jhi - Jlo + 1;
        const int qd = u % P;
        u /= P;
        const int dg = u % ngrp;
        u /= ngrp;
        int o, src;
        if constexpr (XCD) {
            const int opq = 8 / nq;  // octants per queue
            o = (u % opq) * nq + xq;
            src = u / opq;
        } else {
            o = u & 7;
            src = u >> 3;
        }
        const SolveArgs<T> a = at_source(A, src);
        if (a.ctl[g].done) continue;  // this source's group has converged
        const int n = o * D + dg * WPB + w;
        const unsigned stamp = kSignFace ? (unsigned)a.face_par[0] : epoch;
        // sweep geometry: the direction's octant, or the opposite one for the
        // adjoint (the transpose of the DD sweep along W is the sweep along -W)
        const int og = a.rev ? (o ^ 7) : o;
        const int sx = (og & 1) ? -1 : 1, sy = (og & 2) ? -1 : 1, sz = (og & 4) ? -1 : 1;
        const int Jr = Jlo + qd, Kr = d - Jr;
        const int J = sy > 0 ? Jr : NJ - 1 - Jr, K = sz > 0 ? Kr : NK - 1 - Kr;
        // step phase: lane = (j_r, k_r); its physical column (jp, kp)
        const int jr = lane & 7, kr = lane >> 3;
        const int jp = sy > 0 ? jr : 7 - jr, kp = sz > 0 ? kr : 7 - kr;
        const int pl = jp + 8 * kp;
        const int skew = jr + kr;
        const int srcZ = ((lane - 8) & 63) << 2;
        const bool yb = jr == 0, zb = kr == 0, yo = jr == 7, zo = kr == 7;
        const T cx = a.cdir[3 * n], cy = a.cdir[3 * n + 1], cz = a.cdir[3 * n + 2];
        const T csum = cx + cy + cz;
        const long pen = (long)K * NJ + J;
        const Rsrc rPsi = make_rsrc(a.psi + psi_run(pen, a.Nd, n, nx), (unsigned)(nx * RB));
        const Rsrc rSig = SM ? make_rsrc(a.mat + pen * nx * 64, (unsigned)(nx * 64))
                             : make_rsrc(a.sig + pen * nx * 64, (unsigned)(nx * RB));
        // fixed-axis sets, one byte per cell and direction ([Nd][Vp], pencil
        // order): written by kRecord sweeps, read by kTrans sweeps
        constexpr bool kMask = MODE == kRecord || MODE == kTrans;
        const Rsrc rMask = make_rsrc(kMask ? a.mask + (long)n * Vp + pen * nx * 64 : a.mat,
                                     kMask ? (unsigned)(nx * 64) : 0u);
        const int mbase = sx > 0 ? 0 : (nx - 1) * 64, mstep = sx * 64;
        // face words: [direction][pencil][row][8] of Face::BYTES each (the
        // buffers are sized for the widest codec)
        constexpr int FU = Face::BYTES / 4;  // 32-bit units per face value
        unsigned *const fY = (unsigned *)a.faceY, *const fZ = (unsigned *)a.faceZ;
        const long fdir = (long)n * NJ * NK * nx * 8 * FU;
        const long fown = fdir + pen * nx * 8 * FU;
        const bool hasY = Jr > 0, hasZ = Kr > 0;
        const unsigned fbytes = (unsigned)(nx * FB);
        // the last pencil along y (z) has no downstream neighbour there: its
        // outgoing y (z) words would never be read, so they are not stored
        const Rsrc rFYo = make_rsrc(fY + fown, Jr < NJ - 1 ? fbytes : 0u);
        const Rsrc rFZo = make_rsrc(fZ + fown, Kr < NK - 1 ? fbytes : 0u);
        const Rsrc rFYi = make_rsrc(fY + (hasY ? fdir + ((long)K * NJ + (J - sy)) * nx * 8 * FU : 0), hasY ? fbytes : 0);
        const Rsrc rFZi = make_rsrc(fZ + (hasZ ? fdir + ((long)(K - sz) * NJ + J) * nx * 8 * FU : 0), hasZ ? fbytes : 0);
        // Octant-relative row r is physical row sx > 0 ? r : nx-1-r, at byte
        // pbase + r * pstep of the pencil.  For every r outside [0, nx) that
        // offset (plus a lane offset below one row) is negative or past the
        // end, i.e. out of the buffer: loads there read zero and stores are
        // dropped, with no test.
        const int pstep = sx * RB, pbase = sx > 0 ? 0 : (nx - 1) * RB;
        const int fstep = sx * FB, fbase = sx > 0 ? 0 : (nx - 1) * FB;
        const int lofs = lane * (int)sizeof(T);  // load phase: lane = physical column
        // load phase for faces: lane = (row in chunk ro, entry e); Y entries
        // are indexed by kp and used by the lane j_r = 0 with skew k_r, Z
        // entries by jp and used by the lane k_r = 0 with skew j_r
        const int e = lane & 7, ro = lane >> 3;
        const int skY = sz > 0 ? e : 7 - e, skZ = sy > 0 ? e : 7 - e;
        const int eoff = e * (int)Face::BYTES;

        // sigma (SM: material byte) of octant-relative row r at byte sbase + r * sstep
        constexpr int SR = Sig::ROW;
        const int sbase = sx > 0 ? 0 : (nx - 1) * SR, sstep = sx * SR;
        const int slofs = pl * (SR / 64);  // the lane's own column (step phase)
        auto sig_off = [&](int ir0) { return sbase + ir0 * sstep + slofs; };

        T pq[CH];  // psi rows of the next chunk (load phase)
        U32x2 pmt;                 // SM: material bytes of the next chunk (load phase)
        typename Sig::Reg ps[CH];  // !SM: sigma of the lane's column at the current chunk's steps
        unsigned pm[CH];           // kTrans: fixed-axis sets of the lane's cells at the current chunk's steps
        typename Face::Word pfy, pfz;
        auto load_rows = [&](int c) {
            int off = pbase + CH * c * pstep + lofs;
#pragma unroll
            for (int b = 0; b < CH; ++b, off += pstep) pq[b] = buf_load<kPsiAux>(rPsi, (unsigned)off, T());
            const unsigned fo = (unsigned)(fbase + (CH * c + ro) * fstep + eoff);
            Face::template load<kLoadAux>(pfy, rFYi, fo);
            Face::template load<kLoadAux>(pfz, rFZi, fo);
            if constexpr (SM) pmt = load_mat_rows(rSig, c, sx, nx, lane);
        };
        // commit chunk c (rows past the end hold zeros and are never used);
        // face words whose stamp is not yet this sweep's are read again
        auto commit = [&](int c) -> bool {
            const int q0 = (CH * c) % RQ;  // 0, 8 or 16: no wrap inside the chunk
#pragma unroll
            for (int b = 0; b < CH; ++b) sQ[w][q0 + b][lane] = pq[b];
            if constexpr (SM) *(U32x2 *)&sMt[w][q0 + mat_row(sx, lane)][8 * (lane & 7)] = pmt;
            const int r = CH * c + ro;
            const bool valid = r < nx;
            bool okY = !valid || !hasY || Face::ok(pfy, stamp);
            bool okZ = !valid || !hasZ || Face::ok(pfz, stamp);
            int spins = 0;
            bool good = true;
            if (__any(!(okY && okZ))) {
                const unsigned fo = (unsigned)(fbase + r * fstep + eoff);
                do {
                    __builtin_amdgcn_s_sleep(2);
                    if (!okY) {
                        Face::template load<kPollAux>(pfy, rFYi, fo);
                        okY = Face::ok(pfy, stamp);
                    }
                    if (!okZ) {
                        Face::template load<kPollAux>(pfz, rFZi, fo);
                        okZ = Face::ok(pfz, stamp);
                    }
                    if (++spins > a0.sweep_spin_limit || ((spins & 255) == 0 && coherent_load(&ctr[1]))) {
                        atomicMax(&ctr[0], kTicketStop);
                        if constexpr (XCD)
                            for (int q = 0; q < nq; ++q) atomicMax(&ctr[kQueueCtr + q], kTicketStop);
                        coherent_store(&ctr[1], 1);
                        good = false;
                        break;
                    }
                } while (__any(!(okY && okZ)));
            }
            sFYi[w][(r + skY) & (RF - 1)][e] = Face::value(pfy);
            sFZi[w][(r + skZ) & (RF - 1)][e] = Face::value(pfz);
            return good;
        };
        T px = T(0), oy = T(0), oz = T(0);
        // One chunk of CH steps.  The chunk's LDS inputs are read first, the
        // steps run from registers, psi and the face outflows go back to LDS
        // at the end.  Lanes outside 0 <= i_r < nx step too, with no test:
        // before its first row a lane sees zero source, sigma and inflow
        // (zeroed ring slots, out-of-range loads), so it carries zero x
        // inflow into row 0; past the last row its results land only in ring
        // slots and face slots of rows that are never stored.
        auto steps = [&](int c) {
            const int t0 = CH * c, ir0 = t0 - skew;
            int s0 = ir0 % RQ;
            s0 = s0 < 0 ? s0 + RQ : s0;
            const int ft = t0 & (RF - 1);  // 0 or 8
            int sq[CH];
            T q[CH], fy[CH], fz[CH], po[CH], yo_[CH], zo_[CH], sg[CH];
#pragma unroll
            for (int b = 0; b < CH; ++b) {
                sq[b] = s0 + b < RQ ? s0 + b : s0 + b - RQ;
                q[b] = sQ[w][sq[b]][pl];
                fy[b] = sFYi[w][ft + b][kp];
                fz[b] = sFZi[w][ft + b][jp];
                if constexpr (SM) sg[b] = sSigT[sMt[w][sq[b]][pl] & (kSigTab - 1)];
            }
            int so = sig_off(ir0 + CH);
            int mo = mbase + ir0 * mstep + pl;  // kRecord / kTrans: the lane's cell at step b
#pragma unroll
            for (int b = 0; b < CH; ++b, so += sstep, mo += mstep) {
                T iny = lane_shr1(oy);
                T inz = lane_from(oz, srcZ);
                iny = yb ? fy[b] : iny;
                inz = zb ? fz[b] : inz;
                T ox_, oy_, oz_;
                unsigned mk = 0;
                if constexpr (MODE == kTrans) mk = pm[b];
                if constexpr (!SM) sg[b] = Sig::value(ps[b], sSigT);
                po[b] = dd_update<T, MODE>(q[b], sg[b], cx, cy, cz, csum, px, iny, inz, ox_, oy_, oz_, mk);
                if constexpr (MODE == kRecord)
                    __builtin_amdgcn_raw_buffer_store_b8((unsigned char)mk, rMask, mo, 0, 0);
                if constexpr (MODE == kTrans)
                    pm[b] = __builtin_amdgcn_raw_buffer_load_b8(rMask, mo + CH * mstep, 0, 0);  // next chunk
                yo_[b] = oy_;
                zo_[b] = oz_;
                px = ox_;
                oy = oy_;
                oz = oz_;
                if constexpr (!SM) ps[b] = Sig::load(rSig, (unsigned)so);  // the next chunk's sigma
            }
#pragma unroll
            for (int b = 0; b < CH; ++b) sQ[w][sq[b]][pl] = po[b];
            if (yo) {
#pragma unroll
                for (int b = 0; b < CH; ++b) sFYo[w][ft + b][kp] = yo_[b];
            }
            if (zo) {
#pragma unroll
                for (int b = 0; b < CH; ++b) sFZo[w][ft + b][jp] = zo_[b];
            }
        };
        // psi rows 8c-16 .. 8c-9 (slots ((8c-16) mod 24) + b) and face rows
        // 8c-14 .. 8c-7 are complete after chunk c
        auto writeback = [&](int c) {
            const int qw = (CH * c + CH) % RQ;  // (8c - 16) mod 24
            T v[CH];
#pragma unroll
            for (int b = 0; b < CH; ++b) v[b] = sQ[w][qw + b][lane];
            int off = pbase + (CH * c - 16) * pstep + lofs;
#pragma unroll
            for (int b = 0; b < CH; ++b, off += pstep) buf_store<kPsiAux>(rPsi, (unsigned)off, v[b]);
            // Y entry e of row r was made by the lane with skew 7 + skY at
            // step r + 7 + skY (Z likewise)
            const int r = CH * c - 14 + ro;
            const unsigned fo = (unsigned)(fbase + r * fstep + eoff);
            Face::template put<kStoreAux>(rFYo, fo, sFYo[w][(r + 7 + skY) & (RF - 1)][e], stamp);
            Face::template put<kStoreAux>(rFZo, fo, sFZo[w][(r + 7 + skZ) & (RF - 1)][e], stamp);
        };

        const int nchunks = (nx + 15) / CH + 1;
        const int cnext = nchunks > 3 ? nchunks - 3 : 0;  // chunk that takes the next ticket
        // Same issue order as inside the loop (rows, faces, then sigma), so
        // the wait at the loop head can leave the newest loads in flight.
        // rows -14 .. -1 (ring slots 10 .. 23) and the face inflow rings start
        // at zero
#pragma unroll
        for (int s = RQ - 14; s < RQ; ++s) sQ[w][s][lane] = T(0);
        if constexpr (SM) {
#pragma unroll
            for (int s = RQ - 14; s < RQ; ++s) sMt[w][s][lane] = 255;  // the ghost: zero sigma
        }
        sFYi[w][lane >> 2][(lane & 3) * 2] = T(0);
        sFYi[w][lane >> 2][(lane & 3) * 2 + 1] = T(0);
        sFZi[w][lane >> 2][(lane & 3) * 2] = T(0);
        sFZi[w][lane >> 2][(lane & 3) * 2 + 1] = T(0);
        load_rows(0);
        __builtin_amdgcn_sched_barrier(0);
        {
            int so = sig_off(-skew);
            if constexpr (!SM) {
#pragma unroll
                for (int b = 0; b < CH; ++b, so += sstep) ps[b] = Sig::load(rSig, (unsigned)so);
            }
            if constexpr (MODE == kTrans) {
                int mo = mbase - skew * mstep + pl;
#pragma unroll
                for (int b = 0; b < CH; ++b, mo += mstep) pm[b] = __builtin_amdgcn_raw_buffer_load_b8(rMask, mo, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        writeback(-1);  // all out of range: only mirrors the loop's issue pattern
        __builtin_amdgcn_sched_barrier(0);
        for (int c = 0; c < nchunks; ++c) {
            if (!commit(c)) break;  // abort: the block leaves at the next ticket
            if (c == cnext && threadIdx.x == 0) {
                tnext = atomicAdd(tctr, 1);
                have_next = true;
            }
            load_rows(c + 1);
            steps(c);
            writeback(c);
        }
    }
}

template <typename T, int MODE, int WPB, bool SM, bool XCD, bool NT>
__global__ __launch_bounds__(64 * WPB) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && WPB >= 2 ? (WPB >= 10 ? 3 : 4) : 1))) void k_sweep(SolveArgs<T> a0, int g)
{
    sweep_body<T, MODE, WPB, SM, XCD, NT, false>(a0, g);
}

// The sweep of every (problem, source) pair of a fused batch in one launch.
template <typename T, int MODE, int WPB, bool SM, bool NT>
__global__ __launch_bounds__(64 * WPB) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 && WPB >= 2 ? (WPB >= 10 ? 3 : 4) : 1))) void k_sweep_multi(SolveArgs<T> a0, int g)
{
    sweep_body<T, MODE, WPB, SM, false, NT, true>(a0, g);
}

// Asks for every cache line of a kernel's arguments at once (BYTES of them, at
// most 512).  The compiler loads arguments where they are used, each new line a
// miss to a place no cache holds yet (33x21x18 solve 1.42 -> 1.40 ms, 32^3 4.46 ->
// 4.40).  Not for kernels that fill the machine: the moments pass lost by it.
template <int BYTES>
__device__ __forceinline__ void fetch_args()
{
    static_assert(BYTES <= 512, "eight lines");
    typedef const __attribute__((address_space(4))) unsigned *Ptr;
    const Ptr k = (Ptr)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr int N = (BYTES + 63) / 64;
    unsigned x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = k[i < N ? 16 * i : 0];
    asm volatile("" ::"s"(x[0]), "s"(x[1]), "s"(x[2]), "s"(x[3]), "s"(x[4]), "s"(x[5]), "s"(x[6]), "s"(x[7]));
    __builtin_amdgcn_sched_barrier(0);
}

// Tile sweep: the same cell updates as k_sweep with the faces between the
// pencils of a tile kept on chip.
//
// Work item = (octant o, direction, tile (TJ_r, TK_r) of tile_y x tile_z
// pencils, source), swept by a team of tile_y * tile_z waves of one block, one
// pencil each, with the per-wave pipeline of k_sweep.  A pencil's y and z
// outflow is handed to the team's next pencil in LDS; only the faces on the
// rim of the tile go through the stamped face words.  What bounds the sweep
// of a small mesh is the chain of pencils along a diagonal: through memory a
// downstream pencil starts three 8-step chunks plus a store-to-load trip of
// 1-2 us after its upstream one.  In LDS the trip is gone, and the hop is 15
// steps: a lane needs the upstream lane's outflow of seven steps later
// (skews 7 apart, same row), so when a pencil's chunk grid is shifted by one
// step against its upstream neighbour's - the phase p = -(J_r + K_r) mod 8,
// p idle steps before the first row - the outflow of one upstream chunk is
// exactly the inflow of one downstream chunk.  Face values are therefore
// exchanged by step, not by row: ring entry (b, e) of a chunk is what the
// lane of entry e made at the chunk's step b, which is what the downstream
// lane of that entry needs at its own step b.
//
// The teams' waves run free: each takes the team's items in order from a
// small ring of tickets (the leading wave fetches them), starts its pencil as
// soon as its inflow is there and goes straight on to the next item, so a
// team pipelines from item to item with no barrier.  Per link and wave a
// counter of the chunks handed over and one of the chunks consumed (kept for
// the whole launch) order the ring of kTileSlots chunks; one LDS read per
// chunk checks both inflows and both outflow rings.
//
// Tickets go tile diagonal by tile diagonal, so an item's upstream tiles hold
// smaller tickets.  Inside a team a wave waits for its upstream waves' next
// chunk of the same or an earlier item, or for a downstream wave to consume a
// chunk at least kTileSlots behind; in the order (item, chunk + j + k) both
// are smaller, so every wait ends.  All are bounded as in k_sweep.
//
// What bounds it then is one wave's own pace, about 1 us a chunk in FP32 and
// 1.7 us with fixup passes: few waves share a SIMD, so every instruction and
// every LDS trip of a chunk counts.  Hence one LDS trip between the steps of
// two chunks, no branch off the common path, and addresses as immediate
// offsets (64x64x16 S6 G90 solve 87.5 -> 81.9 ms, 40^3 S8 2.00 -> 1.87 ms).  The
// sweep of 64^3 S8 takes 92 us (k_sweep: 146-160), in FP64 144 (202-217).
//
// Global rim words: word (slot, entry) of a pencil face, slot = u mod nx with
// u = row + the entry's skew along the face: a bijection of the nx rows of
// each entry, and a chunk's words are one contiguous run (split where it
// wraps).
constexpr int kTileSlots = 3;  // chunks a handover ring holds: 2 stall on jitter, 4 do not fit 16 FP32 waves
constexpr int kItemRing = 8;   // tickets the leading wave may be ahead of the team's last wave

template <typename T, int MODE, int NW, bool SM, bool NT>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : NW > 8 ? 4 : 3))) void k_sweep_tile(SolveArgs<T> a0, int g)
{
    fetch_args<sizeof(a0) + sizeof(g)>();
    constexpr int kPsiAux = NT ? kNT : 0;
    typedef SigSrc<T, SM> Sig;
    typedef typename FaceCodecSel<T, MODE, false>::type Face;
    constexpr bool kSignFace = std::is_same<Face, SignFace<T>>::value;
    constexpr int RQ = 24, CH = 8, NS = kTileSlots;
    constexpr int RB = 64 * sizeof(T);
    constexpr int FB = 8 * (int)Face::BYTES;
    constexpr unsigned kNone = 0x80000000u;  // an offset outside every buffer
    // psi rows move 16 bytes a lane: LR lanes a row, RI rows an access
    constexpr int LR = RB / 16, RI = 64 / LR, NI = CH / RI, VL = 16 / (int)sizeof(T);
    __shared__ __align__(16) T sQ[NW][RQ][64];
    __shared__ __align__(16) T sF[NW][2 + 2 * NS][8][CH];  // face chunks [entry][step]: y, z inflow from memory; y, z outflow rings
    __shared__ __align__(16) unsigned char sMt[SM ? NW : 1][SM ? RQ : 1][64];  // SM: material byte ring (slots as sQ)
    __shared__ int sCtr[NW][4];  // per wave: y, z chunks handed over; y, z chunks its downstream waves have consumed
    __shared__ int sItem[NW][kItemRing], sPub[NW], sTaken[NW];  // tickets of the team led by the wave; items taken
    __shared__ int sAbort, sSpare[NW];
    __shared__ T sSigT[SM ? kSigTab : 1];
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int TY = a0.tile_y, TZ = a0.tile_z, TW = TY * TZ;
    const int team = w / TW, tw = w - team * TW, lead = team * TW;
    const int ja = tw % TY, ka = tw / TY;
    const int D = a0.D;
    const int NJ = a0.g.NJ, NK = a0.g.NK, nx = a0.g.nx;
    const int NTJ = (NJ + TY - 1) / TY, NTK = (NK + TZ - 1) / TZ;
    int *const ctr = a0.sweep_ctr;
    // Everything the first item needs that does not depend on its ticket is
    // asked for together with the ticket: these loads miss every cache, and
    // one after the other they cost a small mesh more than its steps.  (A
    // launch with nothing to do leaves the ticket unused; the next launch
    // starts from zero.)
    int tnext = 0;
    bool have_next = false;
    // its address is made opaque: the compiler would combine a known-uniform
    // atomic over the lanes, and wait for it on the spot
    int opaque0 = 0;
    asm("" : "+v"(opaque0));
    if (tw == 0 && lead + TW <= NW) {
        if (lane == 0) tnext = atomicAdd(&ctr[opaque0], 1);
        have_next = true;
    }
    const bool once = (long)gridDim.x * (NW / TW) >= a0.sweep_nitems;  // every item is a team's first
    const unsigned epoch = (unsigned)const_load(&ctr[2]), par0 = kSignFace ? (unsigned)const_load(a0.face_par) : 0u;
    const int nitems = a0.sweep_nitems;
    const int ndiag = NTJ + NTK - 1;
    const bool dst_reg = ndiag <= 64;  // lane l holds the first ticket of tile diagonal l
    const int dst = dst_reg && lane < ndiag ? a0.sweep_dstart[lane] : 0;
    double sig_m = 0.0;
    if (SM && (int)threadIdx.x < a0.nmat) sig_m = a0.xs_t[threadIdx.x * a0.G + g];
    bool live = false;
    for (int s = 0; s < a0.S; ++s) live = live || !const_load(&a0.ctl[(long)s * a0.G + g].done);
    if (!live) return;
    if (SM && threadIdx.x < kSigTab) sSigT[threadIdx.x] = (T)sig_m;
    if (threadIdx.x < 4 * NW) (&sCtr[0][0])[threadIdx.x] = 0;
    if (threadIdx.x < NW) {
        sPub[threadIdx.x] = 0;
        sTaken[threadIdx.x] = 0;
    }
    if (threadIdx.x == 0) sAbort = 0;
    __syncthreads();  // the only barrier
    // Never taken: a block is a whole number of teams.  This and the test at the
    // first ticket keep the compiler from merging the code on their two sides,
    // whose schedule the solves feel (33x21x18 1.41 ms, 1.45 without this one;
    // 64x64x16 S6 G90 81.5 ms, 82.0 without the other).
    if (lead + TW > NW) return;

    // waits on LDS state: polled much faster than a face word in memory
    const int lds_limit = a0.sweep_spin_limit < 1024 ? a0.sweep_spin_limit
                          : a0.sweep_spin_limit < (1 << 27) ? a0.sweep_spin_limit * 16 : 0x7FFFFFFF;
    auto abort_all = [&]() {
        if (lane == 0) {
            atomicMax(&ctr[0], kTicketStop);
            coherent_store(&ctr[1], 1);
            __hip_atomic_store(&sAbort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };
    auto lds_get = [&](const int *x) { return __hip_atomic_load(x, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP); };
    // past the limit, or another wave (or another block) gave up
    auto gave_up = [&](int spins, int limit) {
        return spins > limit ||
               ((spins & 63) == 0 && __builtin_amdgcn_readfirstlane(__hip_atomic_load(&sAbort, __ATOMIC_RELAXED,
                                                                                      __HIP_MEMORY_SCOPE_WORKGROUP))) ||
               ((spins & 255) == 0 && __builtin_amdgcn_readfirstlane(coherent_load(&ctr[1])));
    };
    // This wave's links, one lane each: lanes 0 and 1 count the chunks handed
    // over to y and z and watch their consumption, lanes 2 and 3 count the
    // chunks consumed from the upstream y and z waves and watch what those hand
    // over.  (The other lanes repeat lane 0 and pass.)
    const int wy = ja > 0 ? w - 1 : w, wz = ka > 0 ? w - TY : w;
    int *const own = &sCtr[0][0] + 4 * w, *const upy = &sCtr[0][0] + 4 * wy, *const upz = &sCtr[0][0] + 4 * wz;
    int *const watch = lane == 1 ? own + 3 : lane == 2 ? upy : lane == 3 ? upz + 1 : own + 2;
    // (a count that nobody watches goes to the wave's spare word)
    int *const tell = lane == 0 ? own : lane == 1 ? own + 1 : lane == 2 && ja > 0 ? upy + 2
                      : lane == 3 && ka > 0 ? upz + 3 : &sSpare[w];
    const bool inY = ja > 0, inZ = ka > 0;  // inflow from the team's neighbour (a link)
    int done = 0;
    int slot = 0;  // the next ring slot of the lane's link
    const int jr = lane & 7, kr = lane >> 3;
    const int skew = jr + kr;
    const int srcZ = ((lane - 8) & 63) << 2;
    const bool yb = jr == 0, zb = kr == 0, yo = jr == 7, zo = kr == 7;
    const int e = lane & 7, ro = lane >> 3;
    const int lrow = lane / LR, lcol = lane % LR;

    bool good = true;
    for (int seq = 0; good; ++seq) {
        int t = 0;
        if (tw == 0) {
            if (seq >= kItemRing) {  // the ring's oldest ticket must have been taken by every wave
                int spins = 0;
                while (good && __any(lane >= 1 && lane < TW && lds_get(&sTaken[lead + (lane < TW ? lane : 0)]) <= seq - kItemRing)) {
                    __builtin_amdgcn_s_sleep(1);
                    good = !gave_up(++spins, lds_limit);
                }
            }
            if (lane == 0) {
                t = have_next ? tnext : once ? nitems : atomicAdd(&ctr[opaque0], 1);
                sItem[lead][seq & (kItemRing - 1)] = t;
                __hip_atomic_store(&sPub[lead], seq + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            have_next = false;
            t = __builtin_amdgcn_readfirstlane(t);
        } else {
            int spins = 0;
            while (good && __builtin_amdgcn_readfirstlane(lds_get(&sPub[lead])) <= seq) {
                __builtin_amdgcn_s_sleep(1);
                good = !gave_up(++spins, lds_limit);
            }
            t = __builtin_amdgcn_readfirstlane(sItem[lead][seq & (kItemRing - 1)]);
            if (lane == 0) __hip_atomic_store(&sTaken[w], seq + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        if (!good || t >= nitems) break;
        // ticket -> (tile diagonal, position, direction, octant, source)
        int d = 0;
        if (dst_reg) {
            d = __popcll(__ballot(lane >= 1 && lane < ndiag && dst <= t));
        } else {
            int hi = ndiag - 1;
            while (d < hi) {
                const int mid = (d + hi + 1) >> 1;
                if (const_load(&a0.sweep_dstart[mid]) <= t) d = mid;
                else hi = mid - 1;
            }
        }
        int u = t - (dst_reg ? __builtin_amdgcn_readlane(dst, d) : const_load(&a0.sweep_dstart[d]));
        const int Tlo = d - (NTK - 1) > 0 ? d - (NTK - 1) : 0;
        const int Thi = d < NTJ - 1 ? d : NTJ - 1;
        const int P = Thi - Tlo + 1;
        const int TJ = Tlo + u % P;
        u /= P;
        const int dir = u % D;
        u /= D;
        const int o = u & 7, src = u >> 3;
        const int Jr = TJ * TY + ja, Kr = (d - TJ) * TZ + ka;
        if (Jr >= NJ || Kr >= NK) continue;  // a pencil outside the mesh (its links are off)
        const SolveArgs<T> a = at_source(a0, src);
        if (a0.S > 1 && const_load(&a.ctl[g].done)) continue;  // this source's group has converged
        const int n = o * D + dir;
        const unsigned stamp = kSignFace ? (a0.S > 1 ? (unsigned)const_load(a.face_par) : par0) : epoch;
        const int og = a.rev ? (o ^ 7) : o;
        const int sx = (og & 1) ? -1 : 1, sy = (og & 2) ? -1 : 1, sz = (og & 4) ? -1 : 1;
        const int J = sy > 0 ? Jr : NJ - 1 - Jr, K = sz > 0 ? Kr : NK - 1 - Kr;
        const int jp = sy > 0 ? jr : 7 - jr, kp = sz > 0 ? kr : 7 - kr;
        const int pl = jp + 8 * kp;
        const T cx = const_load(&a.cdir[3 * n]), cy = const_load(&a.cdir[3 * n + 1]), cz = const_load(&a.cdir[3 * n + 2]);
        const T csum = cx + cy + cz;
        const long pen = (long)K * NJ + J;
        const Rsrc rPsi = make_uniform_rsrc(a.psi + psi_run(pen, a.Nd, n, nx), (unsigned)(nx * RB));
        const Rsrc rSig = SM ? make_uniform_rsrc(a.mat + pen * nx * 64, (unsigned)(nx * 64))
                             : make_uniform_rsrc(a.sig + pen * nx * 64, (unsigned)(nx * RB));
        constexpr bool kMask = MODE == kRecord || MODE == kTrans;
        const Rsrc rMask = make_uniform_rsrc(kMask ? a.mask + (long)n * a.g.Vp + pen * nx * 64 : a.mat,
                                     kMask ? (unsigned)(nx * 64) : 0u);
        const int mbase = sx > 0 ? 0 : (nx - 1) * 64, mstep = sx * 64;
        // Face words in memory: in from the upstream pencil, out in this
        // pencil's own.  One buffer per axis spans both (the lower pencil
        // first); no face (the mesh boundary, or a link) = offset kNone.
        const bool gY = !inY && Jr > 0, gZ = !inZ && Kr > 0;
        const bool outY = ja < TY - 1 && Jr < NJ - 1, outZ = ka < TZ - 1 && Kr < NK - 1;
        const unsigned fpen = (unsigned)(nx * FB);  // bytes of a pencil face
        const long fdir = (long)n * NJ * NK;        // pencil faces before this direction's
        const Rsrc rFY = make_uniform_rsrc((char *)a.faceY + (fdir + pen - (Jr > 0 && sy > 0 ? 1 : 0)) * fpen,
                                   Jr > 0 ? 2 * fpen : fpen);
        const Rsrc rFZ = make_uniform_rsrc((char *)a.faceZ + (fdir + pen - (Kr > 0 && sz > 0 ? NJ : 0)) * fpen,
                                   Kr > 0 ? (unsigned)(NJ + 1) * fpen : fpen);
        const unsigned inYo = sy > 0 ? 0u : fpen, ownYo = Jr > 0 && sy > 0 ? fpen : 0u;
        const unsigned inZo = sz > 0 ? 0u : NJ * fpen, ownZo = Kr > 0 && sz > 0 ? NJ * fpen : 0u;
        // chunk c holds steps 8c - ph .. 8c - ph + 7; ring slots, prologue
        // rows and the chunk count are those of k_sweep with the ph idle
        // steps as rows before the first (out of every buffer: zero source
        // and inflow)
        const int ph = (-(Jr + Kr)) & 7;
        const int first_out = ph > 0 ? 1 : 0;  // downstream starts after chunk 0's steps when ph > 0
        const int phu = (ph + 1) & 7;          // the upstream pencils' phase
        const int nlink = (nx + phu + 15) / CH + 1 - (phu > 0 ? 1 : 0);  // chunks they hand over
        const int nchunks = (nx + ph + 15) / CH + 1;
        // where the leading wave asks for the team's next ticket
        const int cnext = tw != 0 || once ? -1 : nchunks > 3 ? nchunks - 3 : 0;
        const int pstep = sx * RB;
        int poff = (sx > 0 ? 0 : (nx - 1) * RB) + (lrow - ph) * pstep + lcol * 16;  // next chunk's rows, this lane
        // Face words: this lane moves the words of entry e at step ro of a
        // chunk, i.e. of row u - skew at step u along the face.  They sit in
        // slot u, from slot 0 on again past the end (below 8 rows: in slot
        // row).  Tracked: the rows of the next chunk's inflow words.
        const int skY = sz > 0 ? e : 7 - e, skZ = sy > 0 ? e : 7 - e;
        const bool wrap = nx >= 8;
        int rowY = ro - ph - skY, rowZ = ro - ph - skZ;
        const int thrY = wrap ? nx - skY : nx, thrZ = wrap ? nx - skZ : nx;  // first row of the wrapped part
        const unsigned fcY = (unsigned)((wrap ? skY : 0) * FB + e * (int)Face::BYTES);
        const unsigned fcZ = (unsigned)((wrap ? skZ : 0) * FB + e * (int)Face::BYTES);
        const bool pY = !outY && Jr < NJ - 1, pZ = !outZ && Kr < NK - 1;  // outflow to memory
        // rows that have a word in memory (none where the face is a link's or the mesh's)
        const unsigned ninY = gY ? nx : 0, ninZ = gZ ? nx : 0, noutY = pY ? nx : 0, noutZ = pZ ? nx : 0;
        auto face_off = [&](int row, unsigned rows, int thr, unsigned fc) -> unsigned {
            const unsigned o_ = (unsigned)row * FB + fc - (row >= thr ? fpen : 0u);
            return (unsigned)row < rows ? o_ : kNone;
        };
        constexpr int SR = Sig::ROW;
        const int sstep = sx * SR;
        // sigma of row + ph = r in the lane's own column
        auto sig_off = [&](int r) { return (sx > 0 ? 0 : (nx - 1) * SR) + (r - ph) * sstep + pl * (SR / 64); };

        U4 pq[NI];                 // psi rows of the next chunk
        U32x2 pmt;                 // SM: material bytes of the next chunk
        typename Sig::Reg ps[CH];  // !SM: sigma of the lane's column at the current chunk's steps
        unsigned pm[CH];           // kTrans: fixed-axis sets of the lane's cells at the current chunk's steps
        typename Face::Word pfy, pfz;
        unsigned offy = kNone, offz = kNone;
        // rows and inflow words of the next chunk (poff, uin), which starts at row r0
        auto load_rows = [&](int r0) {
#pragma unroll
            for (int i = 0; i < NI; ++i)
                pq[i] = __builtin_amdgcn_raw_buffer_load_b128(rPsi, (unsigned)(poff + i * RI * pstep), 0, kPsiAux);
            offy = face_off(rowY, ninY, thrY, fcY + inYo);
            offz = face_off(rowZ, ninZ, thrZ, fcZ + inZo);
            Face::template load<kSC1>(pfy, rFY, offy);
            Face::template load<kSC1>(pfz, rFZ, offz);
            if constexpr (SM) {
                const int row0 = sx > 0 ? r0 : nx - 8 - r0;
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(rSig, (unsigned)(row0 * 64 + 8 * lane), 0, 0);
                pmt = U32x2{v[0], v[1]};
            }
        };
        // the outflow words of one chunk (dropped off the tile's rim): what
        // its step b made is used downstream at step b - 7
        auto put_faces = [&](int back, T fwy, T fwz) {  // of the chunk that starts `back` rows before rowY, rowZ
            const unsigned oy_ = face_off(rowY - back - 7, noutY, thrY, fcY + ownYo);
            const unsigned oz_ = face_off(rowZ - back - 7, noutZ, thrZ, fcZ + ownZo);
            Face::template put<kSC1>(rFY, oy_, fwy, stamp);
            Face::template put<kSC1>(rFZ, oz_, fwz, stamp);
        };
        // psi rows of the ring from slot qw on, of the chunk four before poff
        U4 wb[NI];
        auto get_rows = [&](int qw) {
#pragma unroll
            for (int i = 0; i < NI; ++i) wb[i] = *(const U4 *)&sQ[w][qw + i * RI + lrow][lcol * VL];
        };
        auto put_rows = [&]() {
#pragma unroll
            for (int i = 0; i < NI; ++i)
                __builtin_amdgcn_raw_buffer_store_b128(wb[i], rPsi, (unsigned)(poff + (i * RI - 4 * CH) * pstep), 0, kPsiAux);
        };
        auto commit = [&](int q0) {
#pragma unroll
            for (int i = 0; i < NI; ++i) *(U4 *)&sQ[w][q0 + i * RI + lrow][lcol * VL] = pq[i];
            if constexpr (SM) {  // as byte offsets into the sigma table
                constexpr unsigned kSh = sizeof(T) == 4 ? 2 : 3;
                *(U32x2 *)&sMt[w][q0 + mat_row(sx, lane)][8 * (lane & 7)] =
                    U32x2{(pmt[0] & 0x1F1F1F1Fu) << kSh, (pmt[1] & 0x1F1F1F1Fu) << kSh};
            }
            // (out of range reads as zero: the mesh boundary's inflow, and what
            // a link leaves unused)
            bool badY = offy != kNone & !Face::ok(pfy, stamp), badZ = offz != kNone & !Face::ok(pfz, stamp);
            if (__builtin_expect(__any(badY | badZ), 0)) {
                int spins = 0;
                do {
                    __builtin_amdgcn_s_sleep(1);
                    if (badY) {
                        Face::template load<kVolatileSC1>(pfy, rFY, offy);
                        badY = !Face::ok(pfy, stamp);
                    }
                    if (badZ) {
                        Face::template load<kVolatileSC1>(pfz, rFZ, offz);
                        badZ = !Face::ok(pfz, stamp);
                    }
                    good = good && !gave_up(++spins, a0.sweep_spin_limit);
                } while (good && __any(badY | badZ));
            }
            sF[w][0][e][ro] = Face::value(pfy);
            sF[w][1][e][ro] = Face::value(pfz);
        };
        T px = T(0), oy = T(0), oz = T(0);
        // ring slot of the lane's row at the next chunk's step 0; its psi (and
        // material) entry there, and where slot 0 follows slot RQ - 1: entry b
        // of a chunk is b rows on from one of the two, so a step's address is
        // one select and an immediate offset
        int s0 = skew ? RQ - skew : 0;
        char *const qcol = (char *)&sQ[w][0][pl];
        unsigned char *const mcol = &sMt[SM ? w : 0][0][SM ? pl : 0];

        // rows -14 .. -1 (and two slots more): zero source, zero sigma
#pragma unroll
        for (int i = 0; i < 16 * RB / 1024; ++i) ((U4 *)&sQ[w][RQ - 16][0])[i * 64 + lane] = U4{0, 0, 0, 0};
        if constexpr (SM) {
            constexpr unsigned kZ = (kSigTab - 1) * sizeof(T) * 0x01010101u;
            ((U4 *)&sMt[w][RQ - 16][0])[lane] = U4{kZ, kZ, kZ, kZ};
        }
        load_rows(-ph);
        __builtin_amdgcn_sched_barrier(0);
        {
            int so = sig_off(-skew);
            if constexpr (!SM) {
#pragma unroll
                for (int b = 0; b < CH; ++b, so += sstep) ps[b] = Sig::load(rSig, (unsigned)so);
            }
            if constexpr (MODE == kTrans) {
                int mo = mbase - (skew + ph) * mstep + pl;
#pragma unroll
                for (int b = 0; b < CH; ++b, mo += mstep) pm[b] = __builtin_amdgcn_raw_buffer_load_b8(rMask, mo, 0, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // chunks c in [link_lo, link_hi) count on this lane's link
        const int link_lo = lane == 2 || lane == 3 ? 0 : first_out;
        const int link_hi = lane == 1 ? (outZ ? nchunks : 0) : lane == 2 ? (inY ? nlink : 0)
                            : lane == 3 ? (inZ ? nlink : 0) : (outY ? nchunks : 0);
        // A wave that runs alone on its SIMD waits out every LDS trip, so a
        // chunk has one: between two chunks' steps all LDS accesses are
        // issued in a row, each in its place (the LDS keeps a wave's order):
        // outflow and the counter that hands it over, finished rows, new rows,
        // the next chunk's inputs, the upstream counter and the inflow it
        // vouches for.  Loads and stores to memory are issued behind them.
        int q0 = 0;                    // ring slot of the chunk's first new row
        int spy = 0, spz = 0;          // the chunk's outflow slots
        const T *fyr, *fzr;            // its inflow
        T q[CH], sg[CH], fy[CH], fz[CH];
        char *qb[CH];
        int seen;
        // (16 waves of a block have too few registers to hold them early)
        constexpr bool kEarly = NW <= 8;
        auto get_inflow = [&]() {
            seen = __hip_atomic_load(watch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
            for (int i = 0; i < CH / VL; ++i) {
                *(U4 *)&fy[i * VL] = *(const U4 *)&fyr[i * VL];
                *(U4 *)&fz[i * VL] = *(const U4 *)&fzr[i * VL];
            }
        };
        // the inputs of chunk c out of the rings, and the loads of chunk c + 1
        auto enter = [&](int c) {
            commit(q0);
            {
                char *const qa = qcol + s0 * RB, *const qw_ = qa - RQ * RB;
                const unsigned char *const ma = mcol + s0 * 64, *const mw = ma - RQ * 64;
                unsigned mb[CH];
#pragma unroll
                for (int b = 0; b < CH; ++b) {
                    const bool in = s0 < RQ - b;
                    qb[b] = in ? qa : qw_;
                    if constexpr (SM) mb[b] = (in ? ma : mw)[b * 64];
                }
#pragma unroll
                for (int b = 0; b < CH; ++b) q[b] = *(const T *)(qb[b] + b * RB);
                spy = __builtin_amdgcn_readlane(slot, 0);
                spz = __builtin_amdgcn_readlane(slot, 1);
                const int scy = __builtin_amdgcn_readlane(slot, 2), scz = __builtin_amdgcn_readlane(slot, 3);
                fyr = inY ? sF[wy][2 + scy][kp] : sF[w][0][kp];
                fzr = inZ ? sF[wz][2 + NS + scz][jp] : sF[w][1][jp];
                if constexpr (kEarly) get_inflow();
                if constexpr (SM) {
#pragma unroll
                    for (int b = 0; b < CH; ++b) sg[b] = *(const T *)((const char *)sSigT + mb[b]);
                }
            }
            if (__builtin_expect(c == cnext, 0)) {
                if (lane == 0) tnext = atomicAdd(&ctr[opaque0], 1);
                have_next = true;
            }
            poff += CH * pstep;
            rowY += CH;
            rowZ += CH;
            load_rows(CH * (c + 1) - ph);
        };
        // (The stores, here all out of range, mirror the loop's issue order,
        // so that the wait for the loads can leave the newest in flight.)
        put_faces(64, T(0), T(0));
        get_rows(0);
        enter(0);
        put_rows();
        T inz = T(0);
        // one way out, at the end of the body (a chunk whose wait gave up runs
        // on over garbage; the launch is reported as failed): with another the
        // compiler would wait in the loop for the newest stores
        for (int c = 0; good && c < nchunks; ++c) {
            // inflow chunks there, outflow slots free
            const int step_ = c >= link_lo && c < link_hi ? 1 : 0;
            const int want = done + (lane == 2 || lane == 3 ? step_ : 1 - NS);
            if constexpr (!kEarly) get_inflow();
            if (__builtin_expect(__any(seen < want), 0)) {
                int spins = 0;
                do {
                    __builtin_amdgcn_s_sleep(1);
                    get_inflow();
                    good = good && !gave_up(++spins, lds_limit);
                } while (good && __any(seen < want));
            }
            T po[CH], yo_[CH], zo_[CH];
            const int ir0 = CH * c - skew;  // row + ph at step 0 of the chunk
            int so = sig_off(ir0 + CH);
            int mo = mbase + (ir0 - ph) * mstep + pl;
#pragma unroll
            for (int b = 0; b < CH; ++b, so += sstep, mo += mstep) {
                T iny = lane_shr1(oy);
                iny = yb ? fy[b] : iny;
                inz = zb ? fz[b] : inz;
                T ox_, oy_, oz_, inz_next;
                unsigned mk = 0;
                if constexpr (MODE == kTrans) mk = pm[b];
                if constexpr (!SM) sg[b] = Sig::value(ps[b], sSigT);
                po[b] = dd_update<T, MODE>(q[b], sg[b], cx, cy, cz, csum, px, iny, inz, ox_, oy_, oz_, mk,
                                           [&](T z) { inz_next = lane_from(z, srcZ); });
                if constexpr (MODE == kRecord)
                    __builtin_amdgcn_raw_buffer_store_b8((unsigned char)mk, rMask, mo, 0, 0);
                if constexpr (MODE == kTrans)
                    pm[b] = __builtin_amdgcn_raw_buffer_load_b8(rMask, mo + CH * mstep, 0, 0);
                yo_[b] = oy_;
                zo_[b] = oz_;
                px = ox_;
                oy = oy_;
                oz = oz_;
                inz = inz_next;
                if constexpr (!SM) ps[b] = Sig::load(rSig, (unsigned)so);
            }
            if (yo) {
#pragma unroll
                for (int i = 0; i < CH / VL; ++i) *(U4 *)&sF[w][2 + spy][kp][i * VL] = *(U4 *)&yo_[i * VL];
            }
            if (zo) {
#pragma unroll
                for (int i = 0; i < CH / VL; ++i) *(U4 *)&sF[w][2 + NS + spz][jp][i * VL] = *(U4 *)&zo_[i * VL];
            }
            // hand the outflow over and free the inflow before anything else
            done += step_;
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __hip_atomic_store(tell, done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            const T fwy = sF[w][2 + spy][e][ro], fwz = sF[w][2 + NS + spz][e][ro];
#pragma unroll
            for (int b = 0; b < CH; ++b) *(T *)(qb[b] + b * RB) = po[b];
            put_faces(CH, fwy, fwz);
            // psi rows 8c-16 .. 8c-9 (counted with the idle steps) are
            // complete, and go back
            q0 = q0 == RQ - CH ? 0 : q0 + CH;
            get_rows(q0);
            slot += step_;
            slot = slot == NS ? 0 : slot;
            s0 = s0 + CH < RQ ? s0 + CH : s0 + CH - RQ;
            enter(c + 1);
            put_rows();
        }
    }
    if (!good) abort_all();
}

// After a sweep that no moments pass follows (which does the same): the
// counter block ready for the next sweep (sweep_counters_next) and, for
// sign-parity faces, the parity of every source that ran (its group had not
// converged) flipped, so that its next sweep rejects these words.
__global__ void k_sweep_after(int *ctr, const Ctl *ctl, int G, int g, int S, int *par, int flip)
{
    const int s = threadIdx.x;
    sweep_counters_next(ctr, s);
    if (flip && s < S && !ctl[(long)s * G + g].done) par[s] ^= 1;
}

// The XCD each workgroup runs on (hardware register XCC_ID), for the
// runtime's check of the workgroup-to-XCD mapping before it uses per-XCD
// queues.
__global__ void k_xcc_probe(int *out, int n)
{
    if (threadIdx.x == 0 && (int)blockIdx.x < n) out[blockIdx.x] = (int)__builtin_amdgcn_s_getreg((3 << 11) | 20);
}

// Order-independent checksum of n 32-bit words (wrapping sum of the words
// and of their rotations), for comparing two sweeps' angular fluence bit for
// bit.
__global__ void k_checksum(const unsigned *x, long n, unsigned long long *out)
{
    unsigned long long acc = 0;
    for (long i = blockIdx.x * 256L + threadIdx.x; i < n; i += (long)gridDim.x * 256)
        acc += (unsigned long long)x[i] * 0x9E3779B1ull + ((unsigned long long)((unsigned)i * 0x85EBCA6Bu) ^ x[i]);
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & 63) == 0) atomicAdd(out, acc);
}

// After a sweep with per-XCD queues: if some source was live and a queue's
// counter never reached its item count (no block ran on that XCD), the abort
// flag is raised with value 2 and the host reports the launch as failed.
__global__ void k_xcd_drained(const Ctl *ctl, int G, int g, int S, int *ctr, int nq, int nitems_q)
{
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    bool live = false;
    for (int s = 0; s < S; ++s) live = live || !ctl[(long)s * G + g].done;
    bool drained = true;
    for (int q = 0; q < nq; ++q) drained = drained && ctr[kQueueCtr + q] >= nitems_q;
    if (live && !drained) ctr[1] = 2;
}

// Default waves per block (directions of one octant that share a pencil
// item); the runtime may pick another divisor of D by timing.
int sweep_wpb(int D, bool fp64)
{
    if (D % 4 == 0 && !fp64) return 4;
    if (D % 2 == 0) return 2;
    return 1;
}

// Waves per block the sweep is built for (FP64 rows take twice the LDS, so
// its list stops at 6).
#define DSN_WPB_F32(X) X(1) X(2) X(3) X(4) X(5) X(6) X(9) X(10) X(12)
#define DSN_WPB_F64(X) X(1) X(2) X(3) X(4) X(5) X(6)

int sweep_wpb_choices(bool fp64, int *out)
{
    int n = 0;
#define DSN_PUT(W) out[n++] = W;
    if (fp64) {
        DSN_WPB_F64(DSN_PUT)
    } else {
        DSN_WPB_F32(DSN_PUT)
    }
#undef DSN_PUT
    return n;
}

// NT (non-temporal angular fluence) variants for the forward cell modes
template <typename T, int MODE, int WPB>
static const void *sweep_kernel(bool sm, bool nt)
{
    if constexpr (MODE == kDD || MODE == kFixup) {
        if (nt)
            return sm ? (const void *)&k_sweep<T, MODE, WPB, true, false, true>
                      : (const void *)&k_sweep<T, MODE, WPB, false, false, true>;
    }
    return sm ? (const void *)&k_sweep<T, MODE, WPB, true, false, false>
              : (const void *)&k_sweep<T, MODE, WPB, false, false, false>;
}

// Per-XCD-queue variants: FP32 with the fixup, up to four waves per block.
template <typename T>
static const void *sweep_kernel_xcd(int wpb, int mode, bool sm, bool nt)
{
    if constexpr (sizeof(T) == 4) {
        if (mode != kFixup) return nullptr;
#define DSN_XPICK(W)                                                                                  \
    if (wpb == W)                                                                                     \
        return nt ? (sm ? (const void *)&k_sweep<float, kFixup, W, true, true, true>                  \
                        : (const void *)&k_sweep<float, kFixup, W, false, true, true>)                \
                  : (sm ? (const void *)&k_sweep<float, kFixup, W, true, true, false>                 \
                        : (const void *)&k_sweep<float, kFixup, W, false, true, false>);
        DSN_XPICK(1) DSN_XPICK(2) DSN_XPICK(3) DSN_XPICK(4)
#undef DSN_XPICK
    }
    return nullptr;
}

bool sweep_xcd_supported(bool fp64, int mode, int wpb) { return !fp64 && mode == kFixup && wpb >= 1 && wpb <= 4; }

// Tile variants: (teams, r) as the launch shape names them, and the waves of a
// team.  A block holds w teams of 4 waves (r = 2) or of 8 (r = 4); FP64 rows
// take twice the LDS, so its list stops at 8 waves.
#define DSN_TILE_F32(X) X(1, 2) X(1, 4) X(2, 2) X(2, 4)
#define DSN_TILE_F64(X) X(1, 2) X(1, 4)
static int tile_team(bool fp64, int w, int r) { return r == 2 ? 4 : !fp64 && w == 1 ? 16 : 8; }

int sweep_tile_choices(bool fp64, int *w_out, int *r_out)
{
    int n = 0;
#define DSN_PUT2(W, R) w_out[n] = W, r_out[n++] = R;
    if (fp64) {
        DSN_TILE_F64(DSN_PUT2)
    } else {
        DSN_TILE_F32(DSN_PUT2)
    }
#undef DSN_PUT2
    return n;
}

// The tile of a team on an NJ x NK grid of pencils: of the factorings of its
// wave count the one with the fewest tiles, then the fewest tile diagonals
// (hops through memory), then the squarest.
void sweep_tile(bool fp64, int w, int r, int NJ, int NK, int *ty, int *tz)
{
    const int n = tile_team(fp64, w, r);
    long best = -1;
    for (int y = 1; y <= n; ++y) {
        if (n % y) continue;
        const int z = n / y, nj = (NJ + y - 1) / y, nk = (NK + z - 1) / z;
        const long cost = ((long)nj * nk * 4096 + nj + nk) * 64 + (y > z ? y - z : z - y);
        if (best < 0 || cost < best) best = cost, *ty = y, *tz = z;
    }
}

template <typename T, int MODE, int NW>
static const void *sweep_kernel_tile_of(bool sm, bool nt)
{
    if constexpr (MODE == kDD || MODE == kFixup) {
        if (nt)
            return sm ? (const void *)&k_sweep_tile<T, MODE, NW, true, true>
                      : (const void *)&k_sweep_tile<T, MODE, NW, false, true>;
    }
    return sm ? (const void *)&k_sweep_tile<T, MODE, NW, true, false>
              : (const void *)&k_sweep_tile<T, MODE, NW, false, false>;
}

template <typename T, int NW>
static const void *sweep_kernel_tile_nw(int mode, bool sm, bool nt)
{
    switch (mode) {
    case kDD: return sweep_kernel_tile_of<T, kDD, NW>(sm, nt);
    case kFixup: return sweep_kernel_tile_of<T, kFixup, NW>(sm, nt);
    case kRecord: return sweep_kernel_tile_of<T, kRecord, NW>(sm, nt);
    case kTrans: return sweep_kernel_tile_of<T, kTrans, NW>(sm, nt);
    default: return nullptr;
    }
}

// waves of a block of the tile shape (w, r)
static int tile_waves(bool fp64, int w, int r) { return w * tile_team(fp64, w, r); }

template <typename T>
static const void *sweep_kernel_tile(int w, int r, int mode, bool sm, bool nt)
{
    const int nw = tile_waves(sizeof(T) == 8, w, r);
    if (nw == 4) return sweep_kernel_tile_nw<T, 4>(mode, sm, nt);
    if (nw == 8) return sweep_kernel_tile_nw<T, 8>(mode, sm, nt);
    if constexpr (sizeof(T) == 4)
        if (nw == 16) return sweep_kernel_tile_nw<T, 16>(mode, sm, nt);
    return nullptr;
}

bool sweep_tagged_faces(bool fp64, int mode, int wpb, int xcd)
{
    return mode == kDD || mode == kTrans || (xcd > 0 && sweep_xcd_supported(fp64, mode, wpb));
}

template <typename T>
static const void *sweep_kernel_of(int wpb, int mode, bool sm, bool nt)
{
#define DSN_PICK(W)                                           \
    if (wpb == W) {                                           \
        switch (mode) {                                       \
        case kDD: return sweep_kernel<T, kDD, W>(sm, nt);         \
        case kFixup: return sweep_kernel<T, kFixup, W>(sm, nt);   \
        case kRecord: return sweep_kernel<T, kRecord, W>(sm, nt); \
        case kTrans: return sweep_kernel<T, kTrans, W>(sm, nt);   \
        default: return nullptr;                              \
        }                                                     \
    }
    if constexpr (sizeof(T) == 8) {
        DSN_WPB_F64(DSN_PICK)
    } else {
        DSN_WPB_F32(DSN_PICK)
    }
#undef DSN_PICK
    return nullptr;
}

// Fused-batch (several problems per launch) variants: the forward cell
// modes, global queue, up to five waves per block in FP32 and three in FP64
// (every S_N order up to S16 has a divisor of N(N+2)/8 among them).
#define DSN_WPB_MULTI_F32(X) X(1) X(2) X(3) X(4) X(5)
#define DSN_WPB_MULTI_F64(X) X(1) X(2) X(3)

int sweep_multi_choices(bool fp64, int *out)
{
    int n = 0;
#define DSN_PUT(W) out[n++] = W;
    if (fp64) {
        DSN_WPB_MULTI_F64(DSN_PUT)
    } else {
        DSN_WPB_MULTI_F32(DSN_PUT)
    }
#undef DSN_PUT
    return n;
}

template <typename T, int MODE, int WPB>
static const void *sweep_kernel_multi_nt(bool sm, bool nt)
{
    if (nt)
        return sm ? (const void *)&k_sweep_multi<T, MODE, WPB, true, true>
                  : (const void *)&k_sweep_multi<T, MODE, WPB, false, true>;
    return sm ? (const void *)&k_sweep_multi<T, MODE, WPB, true, false>
              : (const void *)&k_sweep_multi<T, MODE, WPB, false, false>;
}

template <typename T>
static const void *sweep_kernel_multi(int wpb, int mode, bool sm, bool nt)
{
    if (mode != kDD && mode != kFixup) return nullptr;
#define DSN_MPICK(W)                                                                                   \
    if (wpb == W)                                                                                      \
        return mode == kDD ? sweep_kernel_multi_nt<T, kDD, W>(sm, nt) : sweep_kernel_multi_nt<T, kFixup, W>(sm, nt);
    if constexpr (sizeof(T) == 8) {
        DSN_WPB_MULTI_F64(DSN_MPICK)
    } else {
        DSN_WPB_MULTI_F32(DSN_MPICK)
    }
#undef DSN_MPICK
    return nullptr;
}

// Resident blocks of the fused-batch sweep (grid size), 0 if not built.
template <typename T>
int sweep_grid_multi(int wpb, int mode, int n_cu)
{
    int per_cu = 1 << 30;
    for (int sm = 0; sm < 2; ++sm) {
        const void *f = sweep_kernel_multi<T>(wpb, mode, sm != 0, false);
        if (!f) return 0;
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, 64 * wpb, 0) != hipSuccess || n < 1) n = 1;
        per_cu = n < per_cu ? n : per_cu;
    }
    return per_cu * n_cu;
}

// One sweep over every (problem, source) pair of a fused batch: a.multi (device
// copy of host_tab) and a.seg set, a.sweep_ctr the batch's own counter block.
// follow: the batch's moments pass comes next; else the counters and each
// problem's face parity are made ready for the next sweep here.
template <typename T>
int launch_sweep_multi(const SolveArgs<T> &a, const SolveArgs<T> *host_tab, int n, int g, hipStream_t s, bool follow,
                       hipEvent_t ev_before, hipEvent_t ev_after)
{
    const void *f = sweep_kernel_multi<T>(a.sweep_wpb, a.sweep_mode, a.sig_from_mat != 0, a.stream_nt != 0);
    if (!f) return 0;
    SolveArgs<T> arg = a;
    int gi = g;
    void *params[2] = {&arg, &gi};
    const unsigned grid = (unsigned)(a.sweep_grid < a.sweep_nitems ? a.sweep_grid : a.sweep_nitems);
    if (ev_before) (void)hipEventRecord(ev_before, s);
    (void)hipLaunchKernel(f, dim3(grid), dim3(64 * a.sweep_wpb), params, 0, s);
    if (ev_after) (void)hipEventRecord(ev_after, s);
    if (!follow)
        for (int q = 0; q < n; ++q) {
            const SolveArgs<T> &b = host_tab[q];
            hipLaunchKernelGGL(k_sweep_after, dim3(1), dim3(64), 0, s, a.sweep_ctr, b.ctl, b.G, g, b.S, b.face_par,
                               a.sweep_mode == kFixup);
        }
    return 1;
}

// A tile wave's z faces, the upstream pencil's and its own, lie in one buffer
// of a row of NJ + 1 pencil faces, with offsets from kNone = 2^31 up outside
// it.  (In FP64 a row that long belongs to a mesh of 100 GB and more.)
bool sweep_tile_addressable(bool fp64, int nx, int NJ)
{
    const long face_row = 8L * (fp64 ? TaggedFace<double>::BYTES : TaggedFace<float>::BYTES);  // the widest codec
    return (NJ + 1L) * nx * face_row <= 1L << 31;
}

// Resident blocks of the tile sweep of shape (w, r) in cell mode `mode` (grid
// size), 0 if there is no such kernel, for a mesh beyond its face offsets or for
// an x extent beyond the shape's range.  The kernel's LDS does not depend on nx;
// the range is the one these shapes are documented and accepted for (nx up to
// 2252, 974 and 335 for w * r = 2, 4 and 8 in FP32, 998 and 359 for 2 and 4 in
// FP64), and pencils sweep longer ones.
template <typename T>
int sweep_grid_tile(int w, int r, int mode, int nx, int NJ, int n_cu)
{
    const int n = w * r, longest = sizeof(T) == 8 ? (n == 2 ? 998 : 359) : n == 2 ? 2252 : n == 4 ? 974 : 335;
    if (nx > longest || !sweep_tile_addressable(sizeof(T) == 8, nx, NJ)) return 0;
    int per_cu = 1 << 30;
    for (int sm = 0; sm < 2; ++sm) {
        const void *f = sweep_kernel_tile<T>(w, r, mode, sm != 0, false);
        if (!f) return 0;
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, 64 * tile_waves(sizeof(T) == 8, w, r), 0) != hipSuccess ||
            n < 1) {
            (void)hipGetLastError();
            return 0;
        }
        per_cu = n < per_cu ? n : per_cu;
    }
    return per_cu * n_cu;
}

// Resident blocks of the sweep kernel with wpb waves per block in cell mode
// `mode` (grid size), 0 if there is no such kernel.
template <typename T>
int sweep_grid(int wpb, int mode, int n_cu)
{
    int per_cu = 1 << 30;
    for (int sm = 0; sm < 2; ++sm) {  // both sigma variants: the smaller residency
        const void *f = sweep_kernel_of<T>(wpb, mode, sm != 0, false);
        if (!f) return 0;
        int n = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, 64 * wpb, 0) != hipSuccess || n < 1) n = 1;
        per_cu = n < per_cu ? n : per_cu;
    }
    return per_cu * n_cu;
}

// Whether a sweep with these arguments leaves sign-parity face words.
template <typename T>
bool sweep_flips_parity(const SolveArgs<T> &a)
{
    return !sweep_tagged_faces(sizeof(T) == 8, a.sweep_mode, a.sweep_wpb, a.sweep_relay > 0 ? 0 : a.sweep_xcd);
}

// Launches the sweep in cell mode a.sweep_mode with a.sweep_wpb waves per
// block (one of the built choices; the runtime never passes another).
// follow: the moments pass of this sweep comes next on the stream and makes the
// counters and the face parity ready for the next sweep, else they are here.
template <typename T>
int launch_sweeps(const SolveArgs<T> &a, int g, hipStream_t s, bool follow, hipEvent_t ev_before, hipEvent_t ev_after)
{
    // tile items, per-XCD queues where such a kernel is built (FP32 fixup
    // sweeps), else pencil items on the global queue
    const bool tile = a.sweep_relay > 0;
    const bool xcd = !tile && a.sweep_xcd > 0 && sweep_xcd_supported(sizeof(T) == 8, a.sweep_mode, a.sweep_wpb);
    const bool nt = a.stream_nt != 0;
    const void *f = tile ? sweep_kernel_tile<T>(a.sweep_wpb, a.sweep_relay, a.sweep_mode, a.sig_from_mat != 0, nt)
                    : xcd ? sweep_kernel_xcd<T>(a.sweep_wpb, a.sweep_mode, a.sig_from_mat != 0, nt)
                          : sweep_kernel_of<T>(a.sweep_wpb, a.sweep_mode, a.sig_from_mat != 0, nt);
    if (!f) return 0;
    unsigned grid = (unsigned)(a.sweep_grid < a.sweep_nitems ? a.sweep_grid : a.sweep_nitems);
    if (xcd)  // a whole number of blocks per XCD, at least one each
        grid = (grid + a.sweep_xcd - 1) / a.sweep_xcd * a.sweep_xcd;
    SolveArgs<T> arg = a;
    if (!xcd) arg.sweep_xcd = 0;
    int waves = a.sweep_wpb;
    if (tile) {
        sweep_tile(sizeof(T) == 8, a.sweep_wpb, a.sweep_relay, a.g.NJ, a.g.NK, &arg.tile_y, &arg.tile_z);
        waves = tile_waves(sizeof(T) == 8, a.sweep_wpb, a.sweep_relay);
    }
    void *params[2] = {&arg, &g};
    if (ev_before) (void)hipEventRecord(ev_before, s);
    (void)hipLaunchKernel(f, dim3(grid), dim3(64 * waves), params, 0, s);
    if (ev_after) (void)hipEventRecord(ev_after, s);
    if (xcd)
        hipLaunchKernelGGL(k_xcd_drained, dim3(1), dim3(64), 0, s, a.ctl, a.G, g, a.S, a.sweep_ctr, a.sweep_xcd,
                           a.sweep_nitems / a.sweep_xcd);
    if (!follow)
        hipLaunchKernelGGL(k_sweep_after, dim3(1), dim3(64), 0, s, a.sweep_ctr, a.ctl, a.G, g, a.S, a.face_par,
                           sweep_flips_parity(a) ? 1 : 0);
    return 1;
}

void launch_xcc_probe(int *out, int n, hipStream_t s)
{
    hipLaunchKernelGGL(k_xcc_probe, dim3(n), dim3(64), 0, s, out, n);
}

void launch_checksum(const void *x, long n_words, unsigned long long *out, hipStream_t s)
{
    hipLaunchKernelGGL(k_checksum, dim3(1024), dim3(256), 0, s, (const unsigned *)x, n_words, out);
}

template int sweep_grid<float>(int, int, int);
template int sweep_grid<double>(int, int, int);
template int sweep_grid_tile<float>(int, int, int, int, int, int);
template int sweep_grid_tile<double>(int, int, int, int, int, int);
template int launch_sweeps<float>(const SolveArgs<float> &, int, hipStream_t, bool, hipEvent_t, hipEvent_t);
template int launch_sweeps<double>(const SolveArgs<double> &, int, hipStream_t, bool, hipEvent_t, hipEvent_t);
template bool sweep_flips_parity<float>(const SolveArgs<float> &);
template bool sweep_flips_parity<double>(const SolveArgs<double> &);
template int sweep_grid_multi<float>(int, int, int);
template int sweep_grid_multi<double>(int, int, int);
template int launch_sweep_multi<float>(const SolveArgs<float> &, const SolveArgs<float> *, int, int, hipStream_t, bool,
                                       hipEvent_t, hipEvent_t);
template int launch_sweep_multi<double>(const SolveArgs<double> &, const SolveArgs<double> *, int, int, hipStream_t, bool,
                                        hipEvent_t, hipEvent_t);

}  // namespace dsn

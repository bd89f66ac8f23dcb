// Device kernels of the indentation solve for gfx950 (CDNA4, wave64).
//
// Data layout in HBM.
//   Topology (shared by every instance of one mesh): nodes numbered by first
//   touch along the tets' Morton order; tets in Morton order, cut into tiles
//   of at most kTileTets tets that touch at most kTileNodes distinct nodes.
//   Per tile: its node list ("entries", global ids). Per tet, in tile order,
//   one record of D_m^-1, V (computed once in FP64) and four 8-bit local node
//   slots. Node -> entry CSR lists for the deterministic gather of tile
//   partial sums.
//   Instance state: node vectors packed xyz (n x 3), tile partial sums per
//   entry, contact blocks per contact-eligible node, FP64 solver scalars.
//
// Per pass a tile block stages its entries' state vectors in LDS, reads each
// tet's record (shared by every job on the mesh, so a tile's records are
// fetched once per XCD and reused from L2 by the other jobs), recomputes F
// from u, accumulates nodal contributions with FP64 LDS atomics and writes
// one partial per entry; node kernels gather those partials. Global memory
// sees no atomics in the solve kernels.
//
// Control: each instance runs a Newton / PCG / line-search state machine on
// the device. The passes write one FP64 partial per block and per reduced
// quantity; a finalize (one wavefront per instance) sums them in a fixed order
// and takes the transition. A solver step is a tile pass, a node pass and a
// finalize; each instance advances by one phase per step (a CG iteration, a
// line-search trial, a Newton init), whatever phase the others are in. The
// team kernel (k_team) runs all steps of all jobs in one launch, teams of
// workgroups meeting at barriers in the L2; the step kernels (k_tile, k_node,
// k_finalize) run one pass of every job per launch and need no cross-block
// synchronisation.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace fem {

constexpr int kBlock = 256;       // 4 wavefronts of 64
constexpr int kWaves = kBlock / 64;
constexpr int kGather = 6;        // node pass: tile entries per node held with the node
static_assert(kGather == 6, "node_ent4 and node_ent2 hold six entries");
constexpr int kTileTets = 512;    // tets per tile (2 per thread)
constexpr int kTileNodes = 256;   // distinct nodes per tile (8-bit local ids)
static_assert(kTileNodes <= kBlock, "the tile passes stage one entry per thread");
constexpr int kDetElemChunk = 128; // deterministic element pass: tets per chunk of contributions
constexpr int kHistSteps = 1024;  // load steps whose status a job records

enum Phase : int {
    PH_IDLE = 0,
    PH_GRAD = 1,      // element pass at u, then Newton init (start of a load step)
    PH_INIT = 2,      // Newton init after an accepted line-search trial
    PH_CG = 3,        // CG iterations
    PH_TRIAL = 4,     // line-search trial: element pass at u + alpha dx
    PH_DONE = 5,      // all load steps taken
    PH_EVAL_GRAD = 6, // diagnostics: gradient at u, then idle
    PH_EVAL_HV = 7,   // diagnostics: q = H z, then idle
    PH_LAG = 8        // node pass forms the friction lag data, then after_lag
};

// Status codes (same values as the C ABI).
enum : int { ST_OK = 0, ST_FLOOR = 1, ST_NOT_CONVERGED = -6, ST_INVERSION = -7 };

// Partial-sum streams of an instance (each red_stride doubles).
// RS_EN: inertial energy of implicit time steps (node blocks). RS_PQN: slot 0
// holds p.q as every node block summed it (written by node block 0), which the
// finalize takes, so the CG decision and the update applied always agree.
enum : int { RS_PQ = 0, RS_RZ, RS_RR, RS_GD, RS_E, RS_MAG, RS_MINJ, RS_GG, RS_IRZ, RS_EN, RS_PQN, RS_COUNT };

struct Indenter {
    int kind;            // 0 sphere, 1 cylinder, 2 box, 3 ring
    double shape[4];
    double R[9];         // row-major, local -> world
    double c[3];
    double k;
};

struct SolveParams {
    double newton_rtol, newton_atol, cg_rtol, cg_eta_max, c1, noise_eps, floor_rtol, eta_power;
    int max_newton, max_cg, block_jacobi, contact_full, max_halvings, pad;
};

// Dynamic state of one instance (device-resident; the host reads it).
struct InstState {
    int phase, step, steps, step_started;
    int newton_it, cg_it, halvings, apply;
    int status, last_status, last_cg, need_gd;   // last_cg: length of the previous CG solve
    double rz, rr, pq, alpha, beta, tol2;
    double E, emag, minJ, gg, r0, gd, alpha_ls;
    double mu, lam, depth;
    double dt, rho;                           // implicit time step (0: quasi-static), density
    double mdt2;                              // rho / dt^2 (0: quasi-static)
    double gbest;                             // smallest |g_free| of the load step so far
    int stall, steps_floor;                   // accepted iterations without halving gbest
    int model;                                // constitutive law (LAW_NH, LAW_CR)
    unsigned launch;                          // the last launch of the team kernel that took the job (0: none)
    double mu_f, eps_f;                       // Coulomb friction coefficient (0: none), slip smoothing length
    double c_lag[3];                          // indenter centre of the friction lag state
    int lag_ok, after_lag;                    // 1: a lag state exists (u at the step start, c_lag);
                                              // the phase that follows PH_LAG
    double c0[3], dir[3];
    Indenter ind;
    // current load step
    int st_newton, st_cg, st_hv, st_grad, st_ls, pad1;
    double st_g0, st_g;
    // whole job
    long long tot_newton, tot_cg, tot_hv, tot_grad, tot_ls;
    int steps_ok, steps_failed, first_fail, pad2;
};

// Per-tet record in tile order: D_m^-1 (row a = shape gradient of local node
// a+1), rest volume and the four 8-bit local node slots, padded to a multiple
// of 16 bytes so a lane fetches its tet with 16-byte loads from one address.
template <typename T> struct TetRec;
template <> struct alignas(16) TetRec<float> {
    float Bm[9];
    float V;
    uint32_t loc;
    uint32_t pad;
};
template <> struct alignas(16) TetRec<double> {
    double Bm[9];
    double V;
    uint32_t loc;
    uint32_t pad[3];
};
static_assert(sizeof(TetRec<float>) == 48 && sizeof(TetRec<double>) == 96, "tet record layout");

// Buffer pointers of the descriptors below. The host fills them as plain
// pointers; kernels read them through a device view (DEV = true, same
// layout) whose pointers are in the global address space, so accesses
// compile to global memory instructions instead of flat ones (a flat
// instruction also counts against the LDS counter, which makes every wait
// for an LDS result wait for the outstanding memory loads as well).
#ifdef __HIP_DEVICE_COMPILE__
template <class U> using glob_ptr = U __attribute__((address_space(1))) *;
#else
template <class U> using glob_ptr = U *;
#endif
template <class U, bool DEV> using buf_ptr = std::conditional_t<DEV, glob_ptr<U>, U *>;

template <typename T, bool DEV = false>
struct Topo {
    int n, m, ntile, nent, nc, ncb;                 // ncb = contact blocks
    int n_free, pad0;                               // nodes 0 .. n_free-1 are free, the rest fixed
    buf_ptr<const int, DEV> tile_tet;               // ntile + 1
    buf_ptr<const int, DEV> tile_ent;               // ntile + 1
    buf_ptr<const int, DEV> ent_node;               // nent: node of each entry (ascending within a tile)
    buf_ptr<const uint8_t, DEV> ent_slot;           // nent: LDS slot of each entry (local id in the tet records)
    buf_ptr<const TetRec<T>, DEV> rec;              // m, tile order
    buf_ptr<const int, DEV> node_ent_off;           // n + 1
    buf_ptr<const int, DEV> node_ent;               // nent
    buf_ptr<const int4, DEV> node_ent4;             // n: each node's first kGather entries (-1 past its last):
    buf_ptr<const int2, DEV> node_ent2;             // four, then two
    buf_ptr<const int, DEV> inc_off;                // nent + 1: each tile entry's incident (tet, slot) pairs
    buf_ptr<const uint16_t, DEV> inc;               // 4 m: (local tet << 2 | slot), ascending tet per entry
    buf_ptr<const uint8_t, DEV> fixed;              // n
    buf_ptr<const int, DEV> cnodes;                 // nc
    buf_ptr<const int, DEV> cidx;                   // n: contact slot or -1
    buf_ptr<const double, DEV> X;                   // n x 3
    buf_ptr<const T, DEV> nvol;                     // n: lumped volume share sum_e V_e / 4
    buf_ptr<const uint8_t, DEV> owner;              // nent: 1 on each node's first entry
    buf_ptr<const int, DEV> tet_id;                 // m: input index of the tet at each tile position
};

template <typename T, bool DEV = false>
struct InstBufs {
    int topo;
    int red_stride;                                 // partial slots per reduction stream
    buf_ptr<T, DEV> u, dx, g, r, z, p, dinv;        // dinv n x 6, others n x 3
    buf_ptr<T, DEV> pg;                             // nent x 9: gradient (3) + node block (6) partials
    buf_ptr<T, DEV> pq;                             // nent x 3: Hv partials
    buf_ptr<T, DEV> cp;                             // nc x 9: contact gradient (3) + block (6)
    buf_ptr<uint8_t, DEV> cact;                     // nc: 1 where that block is nonzero
    buf_ptr<T, DEV> qout;                           // n x 3 (diagnostics)
    buf_ptr<T, DEV> v, ut;                          // n x 3: velocity of the last completed step, inertial predictor
    buf_ptr<double, DEV> fr;                        // nc x 8: friction lag data (w, normal, displacement
                                                    // relative to the indenter since the lag state, pad)
    buf_ptr<double, DEV> red;                       // RS_COUNT x red_stride
    buf_ptr<signed char, DEV> hist;                 // kHistSteps: status of each load step taken (ST_*)
    buf_ptr<InstState, DEV> s;
};

// Device views of descriptors read from device memory.
template <typename T> using TopoD = Topo<T, true>;
template <typename T> using BufsD = InstBufs<T, true>;
template <typename T> __device__ __forceinline__ TopoD<T> dev_view(const Topo<T> &t) {
    return __builtin_bit_cast(TopoD<T>, t);
}
template <typename T> __device__ __forceinline__ BufsD<T> dev_view(const InstBufs<T> &b) {
    return __builtin_bit_cast(BufsD<T>, b);
}

// ---------------------------------------------------------------------------
// Work mapping: blocks are dealt to the 8 XCDs round-robin, so logical work
// item L is given to hardware block (L % per) * 8 + L / per; consecutive work
// items (same tile of consecutive instances) then share an XCD and its L2.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int logical_block() {
    const int per = gridDim.x >> 3;
    const int b = blockIdx.x;
    return (b & 7) * per + (b >> 3);
}

// ---------------------------------------------------------------------------
// Reductions
// ---------------------------------------------------------------------------
// Wavefront reductions with DPP lane moves (vector ALU, no LDS traffic): a
// prefix sum within each row of 16 lanes (row_shr 1, 2, 4, 8), then the row
// totals carried across rows (row_bcast 15 and 31), so lane 63 holds the
// result, which is broadcast. The order is fixed: every wavefront that
// reduces the same values gets the same bits. Lanes without a source take
// the identity (`empty`, as two 32-bit halves).
template <int CTRL, int ROWMASK>
__device__ __forceinline__ double dpp_move(double v, int empty_lo, int empty_hi) {
    const int lo = __builtin_amdgcn_update_dpp(empty_lo, __double2loint(v), CTRL, ROWMASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(empty_hi, __double2hiint(v), CTRL, ROWMASK, 0xf, false);
    return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double lane63(double v) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), 63),
                            __builtin_amdgcn_readlane(__double2loint(v), 63));
}

__device__ __forceinline__ double wave_sum(double v) {
    v += dpp_move<0x111, 0xf>(v, 0, 0);   // row_shr:1
    v += dpp_move<0x112, 0xf>(v, 0, 0);   // row_shr:2
    v += dpp_move<0x114, 0xf>(v, 0, 0);   // row_shr:4
    v += dpp_move<0x118, 0xf>(v, 0, 0);   // row_shr:8
    v += dpp_move<0x142, 0xa>(v, 0, 0);   // row_bcast:15 into rows 1 and 3
    v += dpp_move<0x143, 0xc>(v, 0, 0);   // row_bcast:31 into rows 2 and 3
    return lane63(v);
}

__device__ __forceinline__ double wave_min(double v) {
    const int ilo = 0, ihi = 0x7ff00000;  // +inf
    v = fmin(v, dpp_move<0x111, 0xf>(v, ilo, ihi));
    v = fmin(v, dpp_move<0x112, 0xf>(v, ilo, ihi));
    v = fmin(v, dpp_move<0x114, 0xf>(v, ilo, ihi));
    v = fmin(v, dpp_move<0x118, 0xf>(v, ilo, ihi));
    v = fmin(v, dpp_move<0x142, 0xa>(v, ilo, ihi));
    v = fmin(v, dpp_move<0x143, 0xc>(v, ilo, ihi));
    return lane63(v);
}

template <int NS, bool MIN>
__device__ __forceinline__ void block_reduce(double (&v)[NS], double &mn) {
    __shared__ double lds[kWaves][NS + 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
    for (int i = 0; i < NS; i++) v[i] = wave_sum(v[i]);
    if (MIN) mn = wave_min(mn);
    if (lane == 0) {
#pragma unroll
        for (int i = 0; i < NS; i++) lds[w][i] = v[i];
        if (MIN) lds[w][NS] = mn;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int i = 0; i < NS; i++) {
            double t = lds[0][i];
            for (int k = 1; k < kWaves; k++) t += lds[k][i];
            v[i] = t;
        }
        if (MIN) {
            double t = lds[0][NS];
            for (int k = 1; k < kWaves; k++) t = fmin(t, lds[k][NS]);
            mn = t;
        }
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// Job data that workgroups of one launch exchange (COH): in the persistent
// team kernel other workgroups write the node vectors, tile partials and
// reduction partials that one reads. Stores write through the CU's vector
// cache to its XCD's L2; the sc1 bit makes a load pass that cache by (it reads
// at the L2's rate: 26 TB/s over the chip measured, as without the bit) and
// makes a store go through the L2 to memory, where other XCDs see it. Vectors
// go through raw buffer accesses, whose cache bits are an argument, scalars
// through relaxed agent-scope atomics.
//   kAlone  one kernel per pass: ordinary loads and stores;
//   kXcd    all readers and writers on one XCD: sc1 loads, ordinary stores;
//   kChip   any XCD: sc1 loads and stores.
// ---------------------------------------------------------------------------
enum : int { kAlone = 0, kXcd = 1, kChip = 2 };
constexpr int kAuxSc1 = 16;                // cache-policy argument of the raw buffer loads: sc1
constexpr int kRsrcFlags = 0x00020000;     // raw buffer, 32-bit data format

// N values of type T of vector i in an array of `count` such vectors.
template <int COH, int N, typename T, class Ptr>
__device__ __forceinline__ void ld_vec(Ptr base, int count, int i, T (&out)[N]) {
    if constexpr (COH == kAlone) {
#pragma unroll
        for (int d = 0; d < N; d++) out[d] = base[N * i + d];
    } else {
        constexpr int kWords = N * (int)sizeof(T) / 4;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, count * (kWords * 4), kRsrcFlags);
        const int off = i * (kWords * 4);
        uint32_t w[kWords];
#pragma unroll
        for (int k = 0; k < kWords; k += 4) {
            const int left = kWords - k;
            if (left >= 4) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b128(rs, off + 4 * k, 0, kAuxSc1);
                __builtin_memcpy(w + k, &v, 16);
            } else if (left == 3) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b96(rs, off + 4 * k, 0, kAuxSc1);
                __builtin_memcpy(w + k, &v, 12);
            } else if (left == 2) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, off + 4 * k, 0, kAuxSc1);
                __builtin_memcpy(w + k, &v, 8);
            } else {
                w[k] = __builtin_amdgcn_raw_buffer_load_b32(rs, off + 4 * k, 0, kAuxSc1);
            }
        }
        __builtin_memcpy(out, w, sizeof out);
    }
}

template <int COH, int N, typename T, class Ptr>
__device__ __forceinline__ void st_vec(Ptr base, int count, int i, const T (&v)[N]) {
    if constexpr (COH != kChip) {
#pragma unroll
        for (int d = 0; d < N; d++) base[N * i + d] = v[d];
    } else {
        constexpr int kWords = N * (int)sizeof(T) / 4;
        typedef uint32_t u2 __attribute__((ext_vector_type(2)));
        typedef uint32_t u3 __attribute__((ext_vector_type(3)));
        typedef uint32_t u4 __attribute__((ext_vector_type(4)));
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, count * (kWords * 4), kRsrcFlags);
        const int off = i * (kWords * 4);
        uint32_t w[kWords];
        __builtin_memcpy(w, v, sizeof w);
#pragma unroll
        for (int k = 0; k < kWords; k += 4) {
            const int left = kWords - k;
            if (left >= 4)
                __builtin_amdgcn_raw_buffer_store_b128(u4{w[k], w[k + 1], w[k + 2], w[k + 3]}, rs, off + 4 * k, 0, kAuxSc1);
            else if (left == 3)
                __builtin_amdgcn_raw_buffer_store_b96(u3{w[k], w[k + 1], w[k + 2]}, rs, off + 4 * k, 0, kAuxSc1);
            else if (left == 2)
                __builtin_amdgcn_raw_buffer_store_b64(u2{w[k], w[k + 1]}, rs, off + 4 * k, 0, kAuxSc1);
            else
                __builtin_amdgcn_raw_buffer_store_b32(w[k], rs, off + 4 * k, 0, kAuxSc1);
        }
    }
}

template <int COH, class U> __device__ __forceinline__ void st_one(U *p, U v) {
    if constexpr (COH == kChip)
        __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        *p = v;
}

template <int COH, class Ptr> __device__ __forceinline__ void st_flag(Ptr base, int count, int i, bool v) {
    if constexpr (COH != kChip) {
        base[i] = v ? 1 : 0;
    } else {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, count, kRsrcFlags);
        __builtin_amdgcn_raw_buffer_store_b8((uint8_t)(v ? 1 : 0), rs, i, 0, kAuxSc1);
    }
}

template <int COH, class U> __device__ __forceinline__ U ld_one(const U *p) {
    if constexpr (COH != kAlone)
        return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else
        return *p;
}

template <int COH, class Ptr> __device__ __forceinline__ bool ld_flag(Ptr base, int count, int i) {
    if constexpr (COH == kAlone) {
        return base[i] != 0;
    } else {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, count, kRsrcFlags);
        return __builtin_amdgcn_raw_buffer_load_b8(rs, i, 0, kAuxSc1) != 0;
    }
}

// As ld_vec and ld_flag, and 0 without an access for i < 0.
template <int COH, int N, typename T, class Ptr>
__device__ __forceinline__ void ld_vec_or0(Ptr base, int count, int i, T (&out)[N]) {
    if constexpr (COH == kAlone) {
        ld_vec<COH>(base, count, i >= 0 ? i : 0, out);
#pragma unroll
        for (int d = 0; d < N; d++) out[d] = i >= 0 ? out[d] : (T)0;
    } else {
        ld_vec<COH>(base, count, i, out);   // out of the buffer's range: reads 0
    }
}

template <int COH, class Ptr> __device__ __forceinline__ bool ld_flag_or0(Ptr base, int count, int i) {
    if constexpr (COH == kAlone)
        return i >= 0 && ld_flag<COH>(base, count, i);
    else
        return ld_flag<COH>(base, count, i);
}

// A value that all lanes hold alike, as a scalar: the team kernel keeps a
// job's solver state in LDS, whose loads return vector registers.
template <int COH> __device__ __forceinline__ int uni(int v) { return COH != kAlone ? __builtin_amdgcn_readfirstlane(v) : v; }
template <int COH> __device__ __forceinline__ float uni(float v) {
    return COH != kAlone ? __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v))) : v;
}
template <int COH> __device__ __forceinline__ double uni(double v) {
    return COH != kAlone ? __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(v)),
                                  __builtin_amdgcn_readfirstlane(__double2loint(v)))
               : v;
}

// Wavefront sums / min of nb partials in a fixed order: lane l adds partials
// l, l + 64, ..., then the wavefront tree. Every wavefront that calls it gets
// the same value (finalize kernel; the node pass's p.q, formed by each of its
// wavefronts without a block barrier). The loads of four partials per lane
// and stream go out together (absent ones count 0), so a sum over up to 256
// partials waits for memory once.
template <int COH, int NS>
__device__ __forceinline__ void wave_sums_partials(const double *const (&part)[NS], int nb, double (&sum)[NS]) {
#pragma unroll
    for (int s = 0; s < NS; s++) sum[s] = 0.0;
    for (int b = threadIdx.x & 63; b < nb; b += 256) {
        double a[NS][4];
#pragma unroll
        for (int k = 0; k < 4; k++)
#pragma unroll
            for (int s = 0; s < NS; s++) a[s][k] = b + 64 * k < nb ? ld_one<COH>(part[s] + b + 64 * k) : 0.0;
#pragma unroll
        for (int k = 0; k < 4; k++)
#pragma unroll
            for (int s = 0; s < NS; s++) sum[s] += a[s][k];
    }
#pragma unroll
    for (int s = 0; s < NS; s++) sum[s] = wave_sum(sum[s]);
}

template <int COH = kAlone> __device__ __forceinline__ double wave_sum_partials(const double *part, int nb) {
    const double *const p[1] = {part};
    double v[1];
    wave_sums_partials<COH, 1>(p, nb, v);
    return v[0];
}

template <int COH = kAlone> __device__ __forceinline__ double wave_min_partials(const double *part, int nb) {
    double v = INFINITY;
    for (int b = threadIdx.x & 63; b < nb; b += 64) v = fmin(v, ld_one<COH>(part + b));
    return wave_min(v);
}

// ---------------------------------------------------------------------------
// Scalar helpers
// ---------------------------------------------------------------------------
template <typename T> __device__ __forceinline__ T fma_t(T a, T b, T c);
template <> __device__ __forceinline__ float fma_t<float>(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
template <> __device__ __forceinline__ double fma_t<double>(double a, double b, double c) { return __builtin_fma(a, b, c); }

template <typename T> __device__ __forceinline__ T log1p_t(T x);
template <> __device__ __forceinline__ float log1p_t<float>(float x) { return log1pf(x); }
template <> __device__ __forceinline__ double log1p_t<double>(double x) { return log1p(x); }

template <typename T> __device__ __forceinline__ T abs_t(T x) { return x < (T)0 ? -x : x; }

template <typename T> __device__ __forceinline__ T safe_recip(T d) {
    return d > (T)0 ? (T)1 / d : (d < (T)0 ? (T)1 / -d : (T)1);
}

// z = M^-1 r of one node, in a fixed order of operations: the node pass
// stores z for the tile pass and forms the same bits again from r in the next
// CG update instead of reading it. The Newton init (init) rounds the first
// product of a row, the CG update the second: the first CG iteration of a
// solve re-forms the init's z.
template <typename T> __device__ __forceinline__ void precond(const T M[6], const T r[3], T z[3], bool init) {
    if (init) {
        z[0] = fma_t(M[4], r[2], fma_t(M[3], r[1], M[0] * r[0]));
        z[1] = fma_t(M[5], r[2], fma_t(M[1], r[1], M[3] * r[0]));
        z[2] = fma_t(M[2], r[2], fma_t(M[5], r[1], M[4] * r[0]));
        return;
    }
    z[0] = fma_t(M[4], r[2], fma_t(M[0], r[0], M[3] * r[1]));
    z[1] = fma_t(M[5], r[2], fma_t(M[3], r[0], M[1] * r[1]));
    z[2] = fma_t(M[2], r[2], fma_t(M[4], r[0], M[5] * r[1]));
}

// ---------------------------------------------------------------------------
// Element kinematics from LDS-staged tile data.
// ---------------------------------------------------------------------------
template <typename T>
struct ElemGeo {
    T Bm[9];   // D_m^-1, row a = shape gradient of local node a+1
    T V;
};

__device__ __forceinline__ void unpack_loc(uint32_t w, int l[4]) {
    l[0] = w & 0xff;
    l[1] = (w >> 8) & 0xff;
    l[2] = (w >> 16) & 0xff;
    l[3] = w >> 24;
}

// Rest constants and local node slots of tet k (tile order) from the per-mesh
// records, fetched as whole 16-byte words (fetch_tet) and unpacked once they
// are needed (unpack_tet), so a fetch can be issued ahead of its use.
template <typename T> struct TetWords {
    uint4 w[sizeof(TetRec<T>) / 16];
};

template <typename T>
__device__ __forceinline__ void fetch_tet(const TopoD<T> &tp, int k, TetWords<T> &tw) {
    const uint4 *src = reinterpret_cast<const uint4 *>(tp.rec + k);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(TetRec<T>) / 16); i++) tw.w[i] = src[i];
}

template <typename T>
__device__ __forceinline__ ElemGeo<T> unpack_tet(const TetWords<T> &tw, int l[4]) {
    TetRec<T> r;
    __builtin_memcpy(&r, tw.w, sizeof r);
    ElemGeo<T> g;
#pragma unroll
    for (int c = 0; c < 9; c++) g.Bm[c] = r.Bm[c];
    g.V = r.V;
    unpack_loc(r.loc, l);
    return g;
}

// Hessian-path helpers: the Hessian only steers the Newton direction (the
// solution is fixed by the gradient), so the tangent's ln J and 1/J use a
// short series and the hardware reciprocal instead of the correctly rounded
// library routines; ~1e-7 relative in FP32, ~1e-13 in FP64 for |J - 1| < 1/2.
template <typename T> __device__ __forceinline__ T fast_rcp(T x);
template <> __device__ __forceinline__ float fast_rcp<float>(float x) { return __builtin_amdgcn_rcpf(x); }
template <> __device__ __forceinline__ double fast_rcp<double>(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    return r;
}

// ln(1 + x) = 2 atanh(s), s = x / (2 + x); |s| <= 0.2 for |x| <= 1/2.
template <typename T>
__device__ __forceinline__ T fast_log1p(T x) {
    if (!(x > (T)-0.5 && x < (T)0.5)) return log1p_t(x);
    const T s = x * fast_rcp((T)2 + x);
    const T s2 = s * s;
    T p;
    if (sizeof(T) == 4) {
        p = fma_t(s2, (T)(1.0 / 9.0), (T)(1.0 / 7.0));
        p = fma_t(s2, p, (T)(1.0 / 5.0));
    } else {
        p = fma_t(s2, (T)(1.0 / 21.0), (T)(1.0 / 19.0));
        p = fma_t(s2, p, (T)(1.0 / 17.0));
        p = fma_t(s2, p, (T)(1.0 / 15.0));
        p = fma_t(s2, p, (T)(1.0 / 13.0));
        p = fma_t(s2, p, (T)(1.0 / 11.0));
        p = fma_t(s2, p, (T)(1.0 / 9.0));
        p = fma_t(s2, p, (T)(1.0 / 7.0));
        p = fma_t(s2, p, (T)(1.0 / 5.0));
    }
    p = fma_t(s2, p, (T)(1.0 / 3.0));
    p = fma_t(s2, p, (T)1);
    return (T)2 * s * p;
}

// Staged node vectors in LDS: kSw values per entry (x, y, z, unused), so a
// node is one aligned 4-vector read.
constexpr int kSw = 4;
template <typename T> using vec4_t = T __attribute__((ext_vector_type(4)));

// The four nodes' staged vectors of one tet, read once into registers.
template <typename T>
__device__ __forceinline__ void load_nodes(const T *sw, const int l[4], T w[4][3]) {
#pragma unroll
    for (int a = 0; a < 4; a++) {
        const vec4_t<T> v = *reinterpret_cast<const vec4_t<T> *>(sw + kSw * l[a]);
        w[a][0] = v.x;
        w[a][1] = v.y;
        w[a][2] = v.z;
    }
}

// G = sum_a (w_{a+1} - w_0) (x) row_a(D_m^-1).
template <typename T>
__device__ __forceinline__ void edge_gradient(const T w[4][3], const T Bm[9], T G[9]) {
    T d[3][3];
#pragma unroll
    for (int a = 0; a < 3; a++)
#pragma unroll
        for (int i = 0; i < 3; i++) d[a][i] = w[a + 1][i] - w[0][i];
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int j = 0; j < 3; j++) G[3 * i + j] = d[0][i] * Bm[j] + d[1][i] * Bm[3 + j] + d[2][i] * Bm[6 + j];
}

// J - 1 = tr G + (sum of principal 2x2 minors of G) + det G, free of the
// cancellation of det(I + G) - 1.
template <typename T>
__device__ __forceinline__ T det_minus_one(const T G[9]) {
    const T trG = G[0] + G[4] + G[8];
    const T m2 = (G[0] * G[4] - G[1] * G[3]) + (G[0] * G[8] - G[2] * G[6]) + (G[4] * G[8] - G[5] * G[7]);
    const T dG = G[0] * (G[4] * G[8] - G[5] * G[7]) - G[1] * (G[3] * G[8] - G[5] * G[6]) + G[2] * (G[3] * G[7] - G[4] * G[6]);
    return trG + m2 + dG;
}

// F^-T = cof(F) / J (FAST: hardware reciprocal, Hessian path only).
template <typename T, bool FAST = false>
__device__ __forceinline__ void inverse_transpose(const T G[9], T J, T FiT[9]) {
    T F[9];
#pragma unroll
    for (int k = 0; k < 9; k++) F[k] = G[k];
    F[0] += (T)1; F[4] += (T)1; F[8] += (T)1;
    const T iJ = FAST ? fast_rcp(J) : (T)1 / J;
    FiT[0] = (F[4] * F[8] - F[5] * F[7]) * iJ;
    FiT[1] = (F[5] * F[6] - F[3] * F[8]) * iJ;
    FiT[2] = (F[3] * F[7] - F[4] * F[6]) * iJ;
    FiT[3] = (F[2] * F[7] - F[1] * F[8]) * iJ;
    FiT[4] = (F[0] * F[8] - F[2] * F[6]) * iJ;
    FiT[5] = (F[1] * F[6] - F[0] * F[7]) * iJ;
    FiT[6] = (F[1] * F[5] - F[2] * F[4]) * iJ;
    FiT[7] = (F[2] * F[3] - F[0] * F[5]) * iJ;
    FiT[8] = (F[0] * F[4] - F[1] * F[3]) * iJ;
}

// ---------------------------------------------------------------------------
// Constitutive laws, per tet from G = F - I (J - 1 and J given).
//   element(): energy density (sum and rounding magnitude of its terms), the
//     first Piola-Kirchhoff stress P, and the node diagonal block of the
//     element's Hessian (or its fixed-rotation part) in the form
//     V (alpha |b|^2 I + beta c c^T), c = Mb b.
//   hessvec(): dP for the perturbation dG.
// LAW_NH, compressible Neo-Hookean: Psi = mu/2 (tr F^T F - 3) - mu ln J +
//   lam/2 ln^2 J. LAW_CR, co-rotational linear elasticity (F = R S):
//   Psi = mu |F - R|^2 + lam/2 (tr S - 3)^2, P = 2 mu (F - R) + lam (tr S - 3) R.
// ---------------------------------------------------------------------------
enum : int { LAW_NH = 0, LAW_CR = 1 };

template <typename T, int LAW> struct Law;

template <typename T> struct Law<T, LAW_NH> {
    __device__ static __forceinline__ void element(const T G[9], T Jm1, T J, T mu, T lam, T &psi, T &mag, T P[9],
                                                   T Mb[9], T &alpha, T &beta) {
        const T lnJ = log1p_t(Jm1);
        const T trG = G[0] + G[4] + G[8];
        T G2 = (T)0;
#pragma unroll
        for (int c = 0; c < 9; c++) G2 += G[c] * G[c];
        const T t1 = (T)0.5 * mu * ((T)2 * trG + G2), t2 = -mu * lnJ, t3 = (T)0.5 * lam * lnJ * lnJ;
        psi = t1 + t2 + t3;
        mag = abs_t(t1) + abs_t(t2) + abs_t(t3);
        inverse_transpose(G, J, Mb);
        // P = mu (F - F^-T) + lam ln J F^-T with F - F^-T = G + F^-T G^T, which
        // keeps full relative precision at small strain.
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const T FG = Mb[3 * i] * G[3 * j] + Mb[3 * i + 1] * G[3 * j + 1] + Mb[3 * i + 2] * G[3 * j + 2];
                P[3 * i + j] = mu * (G[3 * i + j] + FG) + lam * lnJ * Mb[3 * i + j];
            }
        alpha = mu;
        beta = mu + lam - lam * lnJ;
    }

    // dP = mu dG + (mu - lam ln J) (F^-1 dG F^-1)^T + lam tr(F^-1 dG) F^-T
    __device__ static __forceinline__ void hessvec(const T G[9], T Jm1, T J, const T dG[9], T mu, T lam, T dP[9]) {
        const T cc = mu - lam * fast_log1p(Jm1);
        T FiT[9];
        inverse_transpose<T, true>(G, J, FiT);
        // A = F^-1 dG (F^-1 = FiT^T)
        T A[9];
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) A[3 * i + j] = FiT[i] * dG[j] + FiT[3 + i] * dG[3 + j] + FiT[6 + i] * dG[6 + j];
        const T tr = A[0] + A[4] + A[8];
        // (A F^-1)^T_ij = sum_k A_jk FiT_ik
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                const T Mt = A[3 * j] * FiT[3 * i] + A[3 * j + 1] * FiT[3 * i + 1] + A[3 * j + 2] * FiT[3 * i + 2];
                dP[3 * i + j] = mu * dG[3 * i + j] + cc * Mt + lam * tr * FiT[3 * i + j];
            }
    }
};

// Rotation factor of F = I + G (det F > 0) by Newton's iteration for the
// polar decomposition with determinant scaling, X <- (g X + X^-T / g) / 2,
// g = |det X|^(-1/3), to convergence at the working precision.
template <typename T>
__device__ __forceinline__ void polar_rotation(const T G[9], T R[9]) {
#pragma unroll
    for (int c = 0; c < 9; c++) R[c] = G[c];
    R[0] += (T)1;
    R[4] += (T)1;
    R[8] += (T)1;
    const T tol = sizeof(T) == 4 ? (T)8e-7 : (T)4e-15;
    for (int it = 0; it < 12; it++) {
        T C[9];   // cofactors: X^-T = C / det
        C[0] = R[4] * R[8] - R[5] * R[7];
        C[1] = R[5] * R[6] - R[3] * R[8];
        C[2] = R[3] * R[7] - R[4] * R[6];
        C[3] = R[2] * R[7] - R[1] * R[8];
        C[4] = R[0] * R[8] - R[2] * R[6];
        C[5] = R[1] * R[6] - R[0] * R[7];
        C[6] = R[1] * R[5] - R[2] * R[4];
        C[7] = R[2] * R[3] - R[0] * R[5];
        C[8] = R[0] * R[4] - R[1] * R[3];
        const T det = R[0] * C[0] + R[1] * C[1] + R[2] * C[2];
        const float g = exp2f(-log2f((float)abs_t(det)) * (1.0f / 3.0f));
        const T a = (T)0.5 * (T)g, b = (T)0.5 / ((T)g * det);
        T diff = (T)0;
#pragma unroll
        for (int c = 0; c < 9; c++) {
            const T x = a * R[c] + b * C[c];
            diff = fmax(diff, abs_t(x - R[c]));
            R[c] = x;
        }
        if (diff <= tol) break;
    }
}

template <typename T> struct Law<T, LAW_CR> {
    // R, and E = S - I formed without cancellation as (C - I)(S + I)^-1 with
    // C - I = G + G^T + G^T G (C = F^T F, S = R^T F, S + I near 2 I).
    __device__ static __forceinline__ void rotation_strain(const T G[9], T R[9], T E[9]) {
        polar_rotation(G, R);
        T S[9], E2[9];
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) {
                // S = R^T (I + G)
                S[3 * i + j] = R[3 * 0 + i] * G[3 * 0 + j] + R[3 * 1 + i] * G[3 * 1 + j] + R[3 * 2 + i] * G[3 * 2 + j] +
                               R[3 * j + i];
                E2[3 * i + j] = G[3 * i + j] + G[3 * j + i] +
                                (G[3 * 0 + i] * G[3 * 0 + j] + G[3 * 1 + i] * G[3 * 1 + j] + G[3 * 2 + i] * G[3 * 2 + j]);
            }
        // (S + I)^-1, S symmetrised
        T A[9];
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) A[3 * i + j] = (T)0.5 * (S[3 * i + j] + S[3 * j + i]) + (i == j ? (T)1 : (T)0);
        T Ai[9];
        Ai[0] = A[4] * A[8] - A[5] * A[7];
        Ai[1] = A[2] * A[7] - A[1] * A[8];
        Ai[2] = A[1] * A[5] - A[2] * A[4];
        Ai[3] = A[5] * A[6] - A[3] * A[8];
        Ai[4] = A[0] * A[8] - A[2] * A[6];
        Ai[5] = A[2] * A[3] - A[0] * A[5];
        Ai[6] = A[3] * A[7] - A[4] * A[6];
        Ai[7] = A[1] * A[6] - A[0] * A[7];
        Ai[8] = A[0] * A[4] - A[1] * A[3];
        const T id = (T)1 / (A[0] * Ai[0] + A[1] * Ai[3] + A[2] * Ai[6]);
        T Q[9];
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++)
                Q[3 * i + j] = (E2[3 * i] * Ai[j] + E2[3 * i + 1] * Ai[3 + j] + E2[3 * i + 2] * Ai[6 + j]) * id;
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) E[3 * i + j] = (T)0.5 * (Q[3 * i + j] + Q[3 * j + i]);
    }

    __device__ static __forceinline__ void element(const T G[9], T Jm1, T J, T mu, T lam, T &psi, T &mag, T P[9],
                                                   T Mb[9], T &alpha, T &beta) {
        T E[9];
        rotation_strain(G, Mb, E);
        const T trE = E[0] + E[4] + E[8];
        T E2 = (T)0;
#pragma unroll
        for (int c = 0; c < 9; c++) E2 += E[c] * E[c];
        psi = mu * E2 + (T)0.5 * lam * trE * trE;   // |F - R| = |R (S - I)| = |E|
        mag = psi;
        // P = R (2 mu E + lam tr E I)
        T X[9];
#pragma unroll
        for (int c = 0; c < 9; c++) X[c] = (T)2 * mu * E[c];
        X[0] += lam * trE;
        X[4] += lam * trE;
        X[8] += lam * trE;
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++)
                P[3 * i + j] = Mb[3 * i] * X[j] + Mb[3 * i + 1] * X[3 + j] + Mb[3 * i + 2] * X[6 + j];
        alpha = (T)2 * mu;
        beta = lam;
    }

    // R and E = sym(R^T F) - I formed directly: in the tangent E only enters
    // through tr S I - S = (2 + tr E) I - E and lam tr E dR, where its
    // rounding (absolute, about the working precision) is negligible.
    __device__ static __forceinline__ void rotation_strain_direct(const T G[9], T R[9], T E[9]) {
        polar_rotation(G, R);
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = i; j < 3; j++) {
                // S_ij = (R^T (I + G))_ij, symmetrised
                const T sij = R[3 * 0 + i] * G[3 * 0 + j] + R[3 * 1 + i] * G[3 * 1 + j] + R[3 * 2 + i] * G[3 * 2 + j] +
                              R[3 * j + i];
                const T sji = R[3 * 0 + j] * G[3 * 0 + i] + R[3 * 1 + j] * G[3 * 1 + i] + R[3 * 2 + j] * G[3 * 2 + i] +
                              R[3 * i + j];
                const T e = (T)0.5 * (sij + sji) - (i == j ? (T)1 : (T)0);
                E[3 * i + j] = e;
                E[3 * j + i] = e;
            }
    }

    // dP = 2 mu (dG - dR) + lam tr(R^T dG) R + lam tr E dR, dR = R [w]x with
    // (tr S I - S) w = axial(R^T dG - dG^T R).
    __device__ static __forceinline__ void hessvec(const T G[9], T Jm1, T J, const T dG[9], T mu, T lam, T dP[9]) {
        T R[9], E[9];
        rotation_strain_direct(G, R, E);
        T M[9];   // R^T dG
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) M[3 * i + j] = R[i] * dG[j] + R[3 + i] * dG[3 + j] + R[6 + i] * dG[6 + j];
        const T ax[3] = {M[7] - M[5], M[2] - M[6], M[3] - M[1]};
        const T trE = E[0] + E[4] + E[8];
        // K = tr S I - S = (2 + tr E) I - E (symmetric)
        const T k00 = (T)2 + trE - E[0], k11 = (T)2 + trE - E[4], k22 = (T)2 + trE - E[8];
        const T k01 = -E[1], k02 = -E[2], k12 = -E[5];
        const T c00 = k11 * k22 - k12 * k12, c01 = k02 * k12 - k01 * k22, c02 = k01 * k12 - k02 * k11;
        const T c11 = k00 * k22 - k02 * k02, c12 = k01 * k02 - k00 * k12, c22 = k00 * k11 - k01 * k01;
        const T kid = (T)1 / (k00 * c00 + k01 * c01 + k02 * c02);
        const T w0 = (c00 * ax[0] + c01 * ax[1] + c02 * ax[2]) * kid;
        const T w1 = (c01 * ax[0] + c11 * ax[1] + c12 * ax[2]) * kid;
        const T w2 = (c02 * ax[0] + c12 * ax[1] + c22 * ax[2]) * kid;
        const T trM = M[0] + M[4] + M[8];
        // dR = R W, W = [[0, -w2, w1], [w2, 0, -w0], [-w1, w0, 0]]
#pragma unroll
        for (int i = 0; i < 3; i++) {
            const T r0 = R[3 * i], r1 = R[3 * i + 1], r2 = R[3 * i + 2];
            const T dR0 = r1 * w2 - r2 * w1, dR1 = r2 * w0 - r0 * w2, dR2 = r0 * w1 - r1 * w0;
            dP[3 * i + 0] = (T)2 * mu * (dG[3 * i + 0] - dR0) + lam * trM * r0 + lam * trE * dR0;
            dP[3 * i + 1] = (T)2 * mu * (dG[3 * i + 1] - dR1) + lam * trM * r1 + lam * trE * dR1;
            dP[3 * i + 2] = (T)2 * mu * (dG[3 * i + 2] - dR2) + lam * trM * r2 + lam * trE * dR2;
        }
    }
};

// Nodal vectors V S row_a(D_m^-1)^T for nodes a+1; node 0 gets minus the sum.
template <typename T>
__device__ __forceinline__ void element_nodal(const T S[9], const T Bm[9], T V, T f[4][3]) {
#pragma unroll
    for (int a = 0; a < 3; a++)
#pragma unroll
        for (int i = 0; i < 3; i++)
            f[a + 1][i] = V * (S[3 * i] * Bm[3 * a] + S[3 * i + 1] * Bm[3 * a + 1] + S[3 * i + 2] * Bm[3 * a + 2]);
#pragma unroll
    for (int i = 0; i < 3; i++) f[0][i] = -(f[1][i] + f[2][i] + f[3][i]);
}

// ---------------------------------------------------------------------------
// Indenter signed distance, its centre at c, in double precision: value, unit world gradient
// and, inside the indenter, the world Hessian (xx yy zz xy xz yz). Medial
// ties go to the lower axis (x, y, z) and to the radial branch before the
// axial one.
// ---------------------------------------------------------------------------
__device__ inline void sdf_eval(const Indenter &ind, const double c[3], const double x[3], bool want_h, double &phi,
                                double n[3], double Hw[6]) {
    const double *R = ind.R;
    const double d0 = x[0] - c[0], d1 = x[1] - c[1], d2 = x[2] - c[2];
    double q[3];
#pragma unroll
    for (int k = 0; k < 3; k++) q[k] = R[k] * d0 + R[3 + k] * d1 + R[6 + k] * d2;
    double gq[3] = {0.0, 0.0, 0.0};
    double Hq[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    switch (ind.kind) {
    case 0: {
        const double L = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2]);
        phi = L - ind.shape[0];
        if (L > 0.0) {
            const double iL = 1.0 / L;
            gq[0] = q[0] * iL; gq[1] = q[1] * iL; gq[2] = q[2] * iL;
            if (want_h) {
                Hq[0] = (1.0 - gq[0] * gq[0]) * iL; Hq[1] = (1.0 - gq[1] * gq[1]) * iL;
                Hq[2] = (1.0 - gq[2] * gq[2]) * iL; Hq[3] = -gq[0] * gq[1] * iL;
                Hq[4] = -gq[0] * gq[2] * iL; Hq[5] = -gq[1] * gq[2] * iL;
            }
        } else {
            gq[2] = 1.0;
        }
        break;
    }
    case 1: {
        const double a = ind.shape[0], hh = 0.5 * ind.shape[1];
        const double rho = sqrt(q[0] * q[0] + q[1] * q[1]);
        const double ex = rho > 0.0 ? q[0] / rho : 1.0, ey = rho > 0.0 ? q[1] / rho : 0.0;
        const double sz = q[2] >= 0.0 ? 1.0 : -1.0;
        const double dr = rho - a, dz = fabs(q[2]) - hh;
        if (dr > 0.0 && dz > 0.0) {
            phi = sqrt(dr * dr + dz * dz);
            gq[0] = ex * dr / phi; gq[1] = ey * dr / phi; gq[2] = sz * dz / phi;
        } else if (dr > 0.0 || (dz <= 0.0 && dr >= dz)) {
            phi = dr;
            gq[0] = ex; gq[1] = ey;
            if (want_h && phi < 0.0 && rho > 0.0) {
                const double tx = -ey, ty = ex, ir = 1.0 / rho;
                Hq[0] = tx * tx * ir; Hq[1] = ty * ty * ir; Hq[3] = tx * ty * ir;
            }
        } else {
            phi = dz;
            gq[2] = sz;
        }
        break;
    }
    case 2: {
        double o2 = 0.0, dd[3];
        bool outside = false;
#pragma unroll
        for (int i = 0; i < 3; i++) {
            dd[i] = fabs(q[i]) - ind.shape[i];
            if (dd[i] > 0.0) { outside = true; o2 += dd[i] * dd[i]; }
        }
        if (outside) {
            phi = sqrt(o2);
#pragma unroll
            for (int i = 0; i < 3; i++) gq[i] = dd[i] > 0.0 ? (q[i] >= 0.0 ? dd[i] : -dd[i]) / phi : 0.0;
        } else {
            int j = 0;
            if (dd[1] > dd[j]) j = 1;
            if (dd[2] > dd[j]) j = 2;
            phi = dd[j];
            gq[j] = q[j] >= 0.0 ? 1.0 : -1.0;
        }
        break;
    }
    default: {
        const double Rm = ind.shape[0], rm = ind.shape[1];
        const double rho = sqrt(q[0] * q[0] + q[1] * q[1]);
        const double ex = rho > 0.0 ? q[0] / rho : 1.0, ey = rho > 0.0 ? q[1] / rho : 0.0;
        const double wr = rho - Rm, wz = q[2];
        const double L = sqrt(wr * wr + wz * wz);
        phi = L - rm;
        if (L > 0.0) {
            const double cr = wr / L, cz = wz / L;
            gq[0] = cr * ex; gq[1] = cr * ey; gq[2] = cz;
            if (want_h && rho > 0.0) {
                // meridian tangent (curvature 1/L) and hoop direction (cr / rho)
                const double tx = -cz * ex, ty = -cz * ey, tz = cr;
                const double iL = 1.0 / L, kh = cr / rho;
                Hq[0] = tx * tx * iL + ey * ey * kh; Hq[1] = ty * ty * iL + ex * ex * kh;
                Hq[2] = tz * tz * iL; Hq[3] = tx * ty * iL - ex * ey * kh;
                Hq[4] = tx * tz * iL; Hq[5] = ty * tz * iL;
            }
        } else {
            gq[2] = 1.0;
        }
        break;
    }
    }
#pragma unroll
    for (int i = 0; i < 3; i++) n[i] = R[3 * i] * gq[0] + R[3 * i + 1] * gq[1] + R[3 * i + 2] * gq[2];
    if (want_h) {
        const double Hf[9] = {Hq[0], Hq[3], Hq[4], Hq[3], Hq[1], Hq[5], Hq[4], Hq[5], Hq[2]};
        double RH[9], W[9];
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) RH[3 * i + j] = R[3 * i] * Hf[j] + R[3 * i + 1] * Hf[3 + j] + R[3 * i + 2] * Hf[6 + j];
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int j = 0; j < 3; j++) W[3 * i + j] = RH[3 * i] * R[3 * j] + RH[3 * i + 1] * R[3 * j + 1] + RH[3 * i + 2] * R[3 * j + 2];
        Hw[0] = W[0]; Hw[1] = W[4]; Hw[2] = W[8]; Hw[3] = W[1]; Hw[4] = W[2]; Hw[5] = W[5];
    }
}

// ---------------------------------------------------------------------------
// End of a load step (called by the finalising thread): bookkeeping, then the
// next load step's pose c = c0 + depth * step / steps * dir, or done.
// ---------------------------------------------------------------------------
__device__ inline void end_step(InstState *s, signed char *hist, int status) {
    s->last_status = status;
    if (hist && s->step >= 1 && s->step <= kHistSteps) hist[s->step - 1] = (signed char)status;
    s->st_g = sqrt(s->gg);
    s->tot_newton += s->st_newton;
    s->tot_cg += s->st_cg;
    s->tot_hv += s->st_hv;
    s->tot_grad += s->st_grad;
    s->tot_ls += s->st_ls;
    if (status >= ST_OK) {
        s->steps_ok++;
        if (status == ST_FLOOR) s->steps_floor++;
    } else {
        s->steps_failed++;
        if (s->first_fail == 0) s->first_fail = status;
    }
    // the state just reached is the next step's friction lag state
    for (int d = 0; d < 3; d++) s->c_lag[d] = s->ind.c[d];
    s->lag_ok = 1;
    if (s->step >= s->steps) {
        s->phase = PH_DONE;
        return;
    }
    s->step++;
    const double f = s->depth * (double)s->step / (double)s->steps;
    for (int d = 0; d < 3; d++) s->ind.c[d] = s->c0[d] + f * s->dir[d];
    s->phase = s->mu_f > 0.0 ? PH_LAG : PH_GRAD;
    s->after_lag = PH_GRAD;
    s->step_started = 1;
    s->newton_it = 0;
    s->st_newton = s->st_cg = s->st_hv = s->st_grad = s->st_ls = 0;
}

// Block-level partial sums of a work kernel: thread 0 stores them.
template <int COH = kAlone, int NS>
__device__ __forceinline__ void store_partials(double *red, int stride, const int (&streams)[NS], int slot,
                                               double (&v)[NS]) {
    if (threadIdx.x == 0)
#pragma unroll
        for (int i = 0; i < NS; i++) st_one<COH>(red + streams[i] * stride + slot, v[i]);
}

// LDS of a tile block, shared by the two tile paths (doubles): the element
// path keeps 9 FP64 accumulators and one staged vector per entry, the
// Hessian path 3 accumulators and two staged vectors.
// In the deterministic mode (DET) the accumulators are replaced by a buffer of
// one chunk of tets' contributions in the path precision: 9 values per node
// and tet (element path, chunks of kDetElemChunk tets) or 3 (Hessian path,
// chunks of kBlock tets).
template <typename T, bool DET = false>
struct TileLds {
    static constexpr int kVec = kSw * kTileNodes * (int)sizeof(T) / 8;
    static constexpr int kElem = DET ? kVec + kDetElemChunk * 36 * (int)sizeof(T) / 8 : 9 * kTileNodes + kVec;
    static constexpr int kTeamHv = 6 * kTileNodes + 2 * kVec;   // team_hessvec: two halves of sums
    static constexpr int kHv = DET ? 2 * kVec + kBlock * 12 * (int)sizeof(T) / 8 : 3 * kTileNodes + 2 * kVec;
    static constexpr int kDoubles = kElem > kHv ? kElem : kHv;
};

// ---------------------------------------------------------------------------
// Lagged, smoothed Coulomb friction at one contact node, in FP64. The lag
// data fr: w = mu_f k (-phi) and the unit normal n at the lag state, then the
// node's displacement relative to the indenter since the lag state, dd: it
// starts at minus the indenter's translation and accumulates the applied
// Newton increments in FP64 (so the slip keeps full precision on the FP32
// path, where it would otherwise be a difference of two rounded positions).
// With the tangential slip s = (I - n n^T) dd and y = |s|: energy
// w f0(y), f0 = y^2/eps - y^3/(3 eps^2) + eps/3 below y = eps and y above
// (C1), gradient w (f1/y) s, and the node block
// w [(f1/y)(I - n n^T) + (f1' - f1/y)/y^2 s s^T] (xx yy zz xy xz yz), which
// is positive semidefinite; f1 = f0'.
// ---------------------------------------------------------------------------
__device__ inline double friction_eval(const double fr[8], const double dd[3], double eps, double g[3], double H[6]) {
    const double w = fr[0];
    const double nl[3] = {fr[1], fr[2], fr[3]};
    const double dn = dd[0] * nl[0] + dd[1] * nl[1] + dd[2] * nl[2];
    double sv[3];
#pragma unroll
    for (int d = 0; d < 3; d++) sv[d] = dd[d] - dn * nl[d];
    const double y = sqrt(sv[0] * sv[0] + sv[1] * sv[1] + sv[2] * sv[2]);
    double f0, a, b;
    if (y < eps) {
        const double ie = 1.0 / eps;
        f0 = y * y * ie - y * y * y * ie * ie * (1.0 / 3.0) + eps * (1.0 / 3.0);
        a = 2.0 * ie - y * ie * ie;              // f1 / y
        b = y > 0.0 ? -ie * ie / y : 0.0;         // (f1' - f1 / y) / y^2
    } else {
        f0 = y;
        a = 1.0 / y;
        b = -a * a * a;
    }
#pragma unroll
    for (int d = 0; d < 3; d++) g[d] = w * a * sv[d];
    H[0] = w * (a * (1.0 - nl[0] * nl[0]) + b * sv[0] * sv[0]);
    H[1] = w * (a * (1.0 - nl[1] * nl[1]) + b * sv[1] * sv[1]);
    H[2] = w * (a * (1.0 - nl[2] * nl[2]) + b * sv[2] * sv[2]);
    H[3] = w * (-a * nl[0] * nl[1] + b * sv[0] * sv[1]);
    H[4] = w * (-a * nl[0] * nl[2] + b * sv[0] * sv[2]);
    H[5] = w * (-a * nl[1] * nl[2] + b * sv[1] * sv[2]);
    return w * f0;
}

// Friction lag data of one contact node at the start of a load step (node
// pass, phase PH_LAG): the penetration and normal at the current
// displacement u (the previous step's result) against the indenter at its
// previous centre c_lag; the relative displacement starts at minus the
// indenter's translation since, c_lag - c.
__device__ inline void friction_lag(const InstState *s, const double x[3], double fr[8]) {
#pragma unroll
    for (int c = 0; c < 8; c++) fr[c] = 0.0;
    if (s->lag_ok) {
        double phl, nl[3], Hn[6];
        sdf_eval(s->ind, s->c_lag, x, false, phl, nl, Hn);
        if (phl < 0.0) {
            fr[0] = s->mu_f * s->ind.k * (-phl);
#pragma unroll
            for (int d = 0; d < 3; d++) fr[1 + d] = nl[d];
        }
    }
#pragma unroll
    for (int d = 0; d < 3; d++) fr[4 + d] = s->c_lag[d] - s->ind.c[d];
}

// Relative displacement of a contact node for friction, with a trial
// increment.
__device__ inline void friction_rel(const double fr[8], const double inc[3], double dd[3]) {
#pragma unroll
    for (int d = 0; d < 3; d++) dd[d] = fr[4 + d] + inc[d];
}

// ---------------------------------------------------------------------------
// Element + contact pass of one tile block (phases GRAD, EVAL_GRAD, TRIAL at
// u + alpha dx). Tile blocks: energy, magnitude, min J, and per entry
// partials of the gradient and of the 3x3 node diagonal blocks
// V (mu |b|^2 I + (mu + lam - lam ln J) c c^T), c = F^-T b. Contact blocks:
// penalty energy, gradient k phi n and block k n n^T (+ k phi Hess(phi) with
// the exact contact Hessian) per eligible node.
// ---------------------------------------------------------------------------
template <typename T, int LAW, bool DET, int COH = kAlone>
__device__ __forceinline__ void tile_element(const TopoD<T> &tp, const BufsD<T> &B, const InstState *s, int blk,
                                             T alpha, int contact_full, double *pool) {
    const T mu = uni<COH>((T)s->mu), lam = uni<COH>((T)s->lam);
    double acc[3] = {0.0, 0.0, INFINITY};   // energy, magnitude, min J
    if (blk < tp.ntile) {
        double *sa = pool;                                    // 9 per entry, FP64 in both precisions
        T *su = (T *)(pool + (DET ? 0 : 9 * kTileNodes));     // kSw per entry
        T *cf = su + kSw * kTileNodes;                        // DET: 36 per tet of a chunk
        const int t = blk;
        const int e0 = tp.tile_ent[t], ne = tp.tile_ent[t + 1] - e0;
        const int k0 = tp.tile_tet[t], nk = tp.tile_tet[t + 1] - k0;
        // This thread's first tet record is fetched before the staging
        // barrier, so its latency overlaps the staging loads.
        TetWords<T> tw;
        if ((int)threadIdx.x < nk) fetch_tet(tp, k0 + (int)threadIdx.x, tw);
        // entry threadIdx.x (ne <= kTileNodes <= kBlock), staged at its slot
        const int sl = (int)threadIdx.x < ne ? tp.ent_slot[e0 + threadIdx.x] : 0;
        if ((int)threadIdx.x < ne) {
            const int gid = tp.ent_node[e0 + threadIdx.x];
            T uu[3], dd[3] = {(T)0, (T)0, (T)0};
            ld_vec<COH>(B.u, tp.n, gid, uu);
            if (alpha != (T)0) ld_vec<COH>(B.dx, tp.n, gid, dd);
#pragma unroll
            for (int d = 0; d < 3; d++) su[kSw * sl + d] = alpha != (T)0 ? fma_t(alpha, dd[d], uu[d]) : uu[d];
            su[kSw * sl + 3] = (T)0;
            if (!DET)
#pragma unroll
                for (int c = 0; c < 9; c++) sa[9 * sl + c] = 0.0;
        }
        __syncthreads();
        // One tet: its energy into acc, and per node a the gradient (c = 0..2)
        // and diagonal block (c = 3..8) contributions to put(l, a, c, value).
        auto tet = [&](int k, auto &&put) {
            int l[4];
            if (k != (int)threadIdx.x) fetch_tet(tp, k0 + k, tw);
            const ElemGeo<T> geo = unpack_tet(tw, l);
            T wu[4][3];
            load_nodes(su, l, wu);
            T G[9];
            edge_gradient(wu, geo.Bm, G);
            const T Jm1 = det_minus_one(G);
            const T J = (T)1 + Jm1;
            acc[2] = fmin(acc[2], (double)J);
            if (!(J > (T)0)) {
                acc[0] = INFINITY;
                return;
            }
            T psi, mag, Pk[9], FiT[9], kI, kc;   // FiT: the block's c = Mb b
            Law<T, LAW>::element(G, Jm1, J, mu, lam, psi, mag, Pk, FiT, kI, kc);
            acc[0] += (double)(geo.V * psi);
            acc[1] += (double)(geo.V * mag);
            T f[4][3];
            element_nodal(Pk, geo.Bm, geo.V, f);
#pragma unroll
            for (int a = 0; a < 4; a++) {
                put(l, a, 0, f[a][0]);
                put(l, a, 1, f[a][1]);
                put(l, a, 2, f[a][2]);
                T bb[3];
                if (a == 0) {
                    bb[0] = -(geo.Bm[0] + geo.Bm[3] + geo.Bm[6]);
                    bb[1] = -(geo.Bm[1] + geo.Bm[4] + geo.Bm[7]);
                    bb[2] = -(geo.Bm[2] + geo.Bm[5] + geo.Bm[8]);
                } else {
                    bb[0] = geo.Bm[3 * (a - 1)];
                    bb[1] = geo.Bm[3 * (a - 1) + 1];
                    bb[2] = geo.Bm[3 * (a - 1) + 2];
                }
                const T cx = FiT[0] * bb[0] + FiT[1] * bb[1] + FiT[2] * bb[2];
                const T cy = FiT[3] * bb[0] + FiT[4] * bb[1] + FiT[5] * bb[2];
                const T cz = FiT[6] * bb[0] + FiT[7] * bb[1] + FiT[8] * bb[2];
                const T sI = geo.V * kI * (bb[0] * bb[0] + bb[1] * bb[1] + bb[2] * bb[2]);
                const T Vk = geo.V * kc;
                put(l, a, 3, sI + Vk * cx * cx);
                put(l, a, 4, sI + Vk * cy * cy);
                put(l, a, 5, sI + Vk * cz * cz);
                put(l, a, 6, Vk * cx * cy);
                put(l, a, 7, Vk * cx * cz);
                put(l, a, 8, Vk * cy * cz);
            }
        };
        if constexpr (!DET) {
            for (int k = threadIdx.x; k < nk; k += kBlock)
                tet(k, [&](const int *l, int a, int c, T v) { atomicAdd(sa + 9 * l[a] + c, (double)v); });
            __syncthreads();
            if ((int)threadIdx.x < ne) {
                T out[9];
#pragma unroll
                for (int c = 0; c < 9; c++) out[c] = (T)sa[9 * sl + c];
                st_vec<COH>(B.pg, tp.nent, e0 + (int)threadIdx.x, out);
            }
        } else {
            // Deterministic: a chunk of tets stores its contributions, then
            // each entry sums its incident ones in ascending tet order.
            double ga[9] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
            const bool mine = (int)threadIdx.x < ne;
            int ip = mine ? tp.inc_off[e0 + threadIdx.x] : 0;
            const int ie = mine ? tp.inc_off[e0 + threadIdx.x + 1] : 0;
            for (int c0 = 0; c0 < nk; c0 += kDetElemChunk) {
                const int k = c0 + (int)threadIdx.x;
                if ((int)threadIdx.x < kDetElemChunk && k < nk) {
                    T *dst = cf + 36 * threadIdx.x;
#pragma unroll
                    for (int q = 0; q < 36; q++) dst[q] = (T)0;
                    tet(k, [&](const int *, int a, int c, T v) { dst[9 * a + c] = v; });
                }
                __syncthreads();
                for (; ip < ie; ip++) {
                    const int code = tp.inc[ip];
                    if ((code >> 2) >= c0 + kDetElemChunk) break;
                    const T *src = cf + 36 * ((code >> 2) - c0) + 9 * (code & 3);
#pragma unroll
                    for (int c = 0; c < 9; c++) ga[c] += (double)src[c];
                }
                __syncthreads();
            }
            if (mine)
#pragma unroll
                for (int c = 0; c < 9; c++) B.pg[9 * (e0 + threadIdx.x) + c] = (T)ga[c];
        }
    } else {
        const int j = (blk - tp.ntile) * kBlock + threadIdx.x;
        if (j < tp.nc) {
            const int i = tp.cnodes[j];
            double x[3];
            T ui[3], di[3] = {(T)0, (T)0, (T)0};
            ld_vec<COH>(B.u, tp.n, i, ui);
            if (alpha != (T)0) ld_vec<COH>(B.dx, tp.n, i, di);
#pragma unroll
            for (int d = 0; d < 3; d++) {
                x[d] = tp.X[3 * i + d] + (double)(alpha != (T)0 ? fma_t(alpha, di[d], ui[d]) : ui[d]);
            }
            double phi, nv[3], Hs[6];
            sdf_eval(s->ind, s->ind.c, x, contact_full != 0, phi, nv, Hs);
            double od[9];
#pragma unroll
            for (int c = 0; c < 9; c++) od[c] = 0.0;
            if (phi < 0.0) {
                const double kp = s->ind.k;
                const double ec = 0.5 * kp * phi * phi;
                acc[0] += ec;
                acc[1] += ec;
#pragma unroll
                for (int d = 0; d < 3; d++) od[d] = kp * phi * nv[d];
                const double nn[6] = {nv[0] * nv[0], nv[1] * nv[1], nv[2] * nv[2], nv[0] * nv[1], nv[0] * nv[2], nv[1] * nv[2]};
#pragma unroll
                for (int c = 0; c < 6; c++) od[3 + c] = kp * (nn[c] + (contact_full ? phi * Hs[c] : 0.0));
            }
            if (s->mu_f > 0.0) {
                double fl[8];
                ld_vec<COH>(B.fr, tp.nc, j, fl);
                if (fl[0] > 0.0) {
                    double inc[3], dd[3], gf[3], Hf[6];
#pragma unroll
                    for (int d = 0; d < 3; d++) inc[d] = (double)alpha * (double)di[d];
                    friction_rel(fl, inc, dd);
                    const double ef = friction_eval(fl, dd, s->eps_f, gf, Hf);
                    acc[0] += ef;
                    acc[1] += ef;
#pragma unroll
                    for (int d = 0; d < 3; d++) od[d] += gf[d];
#pragma unroll
                    for (int c = 0; c < 6; c++) od[3 + c] += Hf[c];
                }
            }
            // the Hessian-vector passes read a node's contact block only
            // where it is nonzero (most eligible nodes are out of contact)
            bool act = false;
            T out[9];
#pragma unroll
            for (int c = 0; c < 9; c++) {
                out[c] = (T)od[c];
                if (c >= 3) act = act || out[c] != (T)0;
            }
            st_vec<COH>(B.cp, tp.nc, j, out);
            st_flag<COH>(B.cact, tp.nc, j, act);
        }
    }
    double sums[2] = {acc[0], acc[1]};
    double mn = acc[2];
    block_reduce<2, true>(sums, mn);
    double v[3] = {sums[0], sums[1], mn};
    const int streams[3] = {RS_E, RS_MAG, RS_MINJ};
    store_partials<COH>(B.red, B.red_stride, streams, blk, v);
}

// Hessian-vector product of one tet from the staged u and p: its LDS slots,
// nodal vectors f and their p; false (nothing) for an inverted tet.
template <typename T, int LAW>
__device__ __forceinline__ bool tet_hessvec(const TetWords<T> &rec, const T *su, const T *sp, T mu, T lam, int l[4],
                                            T f[4][3], T wp[4][3]) {
    T wu[4][3];
    const ElemGeo<T> geo = unpack_tet(rec, l);
    load_nodes(su, l, wu);
    load_nodes(sp, l, wp);
    T G[9];
    edge_gradient(wu, geo.Bm, G);
    const T Jm1 = det_minus_one(G);
    const T J = (T)1 + Jm1;
    if (!(J > (T)0)) return false;
    T dG[9], dP[9];
    edge_gradient(wp, geo.Bm, dG);
    Law<T, LAW>::hessvec(G, Jm1, J, dG, mu, lam, dP);
    element_nodal(dP, geo.Bm, geo.V, f);
    return true;
}

// Share of contact slot j in p.q: p . (contact block) p.
template <typename T, int COH>
__device__ __forceinline__ double contact_hessvec(const TopoD<T> &tp, const BufsD<T> &B, int j, T beta) {
    if (j >= tp.nc || !ld_flag<COH>(B.cact, tp.nc, j)) return 0.0;
    T c9[9], pp[3], zv[3], pv[3];
    const int i = tp.cnodes[j];
    ld_vec<COH>(B.cp, tp.nc, j, c9);
    ld_vec<COH>(B.p, tp.n, i, pp);
    ld_vec<COH>(B.z, tp.n, i, zv);
    const T *H = c9 + 3;
#pragma unroll
    for (int d = 0; d < 3; d++) pv[d] = fma_t(beta, pp[d], zv[d]);
    const T q0 = H[0] * pv[0] + H[3] * pv[1] + H[4] * pv[2];
    const T q1 = H[3] * pv[0] + H[1] * pv[1] + H[5] * pv[2];
    const T q2 = H[4] * pv[0] + H[5] * pv[1] + H[2] * pv[2];
    return (double)(pv[0] * q0 + pv[1] * q1 + pv[2] * q2);
}

// ---------------------------------------------------------------------------
// Hessian-vector product of one tile block (phases CG, EVAL_HV): q = H p with
// p = z + beta p_prev formed while staging (the node pass forms the same
// value). Per tet, with F recomputed from the staged u:
//   dP = mu dG + (mu - lam ln J) (F^-1 dG F^-1)^T + lam tr(F^-1 dG) F^-T.
// p.q is accumulated element by element (and over contact blocks), so alpha
// is known to the node pass without a pass over q.
// ---------------------------------------------------------------------------
template <typename T, int LAW, bool DET>
__device__ __forceinline__ void tile_hessvec(const TopoD<T> &tp, const BufsD<T> &B, const InstState *s, int blk,
                                             double *pool) {
    const T beta = uni<kAlone>((T)s->beta);
    const T mu = uni<kAlone>((T)s->mu), lam = uni<kAlone>((T)s->lam);
    double acc[1] = {0.0};
    double unused = 0.0;
    if (blk < tp.ntile) {
        double *sa = pool;                                    // 3 per entry, FP64 in both precisions
        T *su = (T *)(pool + (DET ? 0 : 3 * kTileNodes));     // kSw per entry
        T *sp = su + kSw * kTileNodes;                        // kSw per entry
        T *cf = sp + kSw * kTileNodes;                        // DET: 12 per tet of a chunk
        const int t = blk;
        const int e0 = tp.tile_ent[t], ne = tp.tile_ent[t + 1] - e0;
        const int k0 = tp.tile_tet[t], nk = tp.tile_tet[t + 1] - k0;
        // Implicit steps add (m_i / dt^2) |p_i|^2 to p.q, taken once per node
        // (on its first entry).
        const double cm = uni<kAlone>(s->mdt2);
        double pq = 0.0;
        // This thread's first tet record is fetched before the staging
        // barrier, so its latency overlaps the staging loads.
        TetWords<T> rec;
        if ((int)threadIdx.x < nk) fetch_tet(tp, k0 + (int)threadIdx.x, rec);
        // entry threadIdx.x (ne <= kTileNodes <= kBlock), staged at its slot
        const int sl = (int)threadIdx.x < ne ? tp.ent_slot[e0 + threadIdx.x] : 0;
        if ((int)threadIdx.x < ne) {
            const int gid = tp.ent_node[e0 + threadIdx.x];
            T pv[3], uv[3], pp[3], zv[3];
            ld_vec<kAlone>(B.u, tp.n, gid, uv);
            ld_vec<kAlone>(B.p, tp.n, gid, pp);
            ld_vec<kAlone>(B.z, tp.n, gid, zv);
#pragma unroll
            for (int d = 0; d < 3; d++) {
                su[kSw * sl + d] = uv[d];
                pv[d] = fma_t(beta, pp[d], zv[d]);
                sp[kSw * sl + d] = pv[d];
                if (!DET) sa[3 * sl + d] = 0.0;
            }
            su[kSw * sl + 3] = (T)0;
            sp[kSw * sl + 3] = (T)0;
            if (cm > 0.0 && tp.owner[e0 + threadIdx.x])
                pq += cm * (double)tp.nvol[gid] *
                      ((double)pv[0] * (double)pv[0] + (double)pv[1] * (double)pv[1] + (double)pv[2] * (double)pv[2]);
        }
        __syncthreads();
        // One tet: its p.q into pq and its nodal vectors to put(l, a, d, value).
        auto tet = [&](int k, auto &&put) {
            int l[4];
            T f[4][3], wp[4][3], e_pq = (T)0;
            if (k != (int)threadIdx.x) fetch_tet(tp, k0 + k, rec);
            if (!tet_hessvec<T, LAW>(rec, su, sp, mu, lam, l, f, wp)) return;
#pragma unroll
            for (int a = 0; a < 4; a++) {
                put(l, a, 0, f[a][0]);
                put(l, a, 1, f[a][1]);
                put(l, a, 2, f[a][2]);
                e_pq += wp[a][0] * f[a][0] + wp[a][1] * f[a][1] + wp[a][2] * f[a][2];
            }
            pq += (double)e_pq;
        };
        if constexpr (!DET) {
            for (int k = threadIdx.x; k < nk; k += kBlock)
                tet(k, [&](const int *l, int a, int d, T v) { atomicAdd(sa + 3 * l[a] + d, (double)v); });
            acc[0] = pq;
            __syncthreads();
            if ((int)threadIdx.x < ne) {
                T out[3];
#pragma unroll
                for (int d = 0; d < 3; d++) out[d] = (T)sa[3 * sl + d];
                st_vec<kAlone>(B.pq, tp.nent, e0 + (int)threadIdx.x, out);
            }
        } else {
            // Deterministic: each chunk of kBlock tets stores its nodal
            // vectors, then each entry sums its incident ones in ascending
            // tet order.
            double qa[3] = {0.0, 0.0, 0.0};
            const bool mine = (int)threadIdx.x < ne;
            int ip = mine ? tp.inc_off[e0 + threadIdx.x] : 0;
            const int ie = mine ? tp.inc_off[e0 + threadIdx.x + 1] : 0;
            for (int c0 = 0; c0 < nk; c0 += kBlock) {
                const int k = c0 + (int)threadIdx.x;
                if (k < nk) {
                    T *dst = cf + 12 * threadIdx.x;
#pragma unroll
                    for (int q = 0; q < 12; q++) dst[q] = (T)0;
                    tet(k, [&](const int *, int a, int d, T v) { dst[3 * a + d] = v; });
                }
                __syncthreads();
                for (; ip < ie; ip++) {
                    const int code = tp.inc[ip];
                    if ((code >> 2) >= c0 + kBlock) break;
                    const T *src = cf + 12 * ((code >> 2) - c0) + 3 * (code & 3);
#pragma unroll
                    for (int d = 0; d < 3; d++) qa[d] += (double)src[d];
                }
                __syncthreads();
            }
            acc[0] = pq;
            if (mine)
#pragma unroll
                for (int d = 0; d < 3; d++) B.pq[3 * (e0 + threadIdx.x) + d] = (T)qa[d];
        }
    } else {
        acc[0] = contact_hessvec<T, kAlone>(tp, B, (blk - tp.ntile) * kBlock + (int)threadIdx.x, beta);
    }
    block_reduce<1, false>(acc, unused);
    const int streams[1] = {RS_PQ};
    store_partials<kAlone>(B.red, B.red_stride, streams, blk, acc);
}

// ---------------------------------------------------------------------------
// Tile pass: one block per (instance, tile or contact block). Each instance's
// blocks take the Hessian-vector path while it is in CG (or EVAL_HV), the
// element path in GRAD, EVAL_GRAD and TRIAL, and return otherwise. The two
// paths share one LDS pool (their register needs are alike, so the union
// does not lower occupancy).
// ---------------------------------------------------------------------------
template <typename T, int LAW, bool DET>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 1 : 3))) void k_tile(const Topo<T> *topos, const InstBufs<T> *bufs, const int2 *work,
                                                 int nwork, const SolveParams *P) {
    __shared__ __attribute__((aligned(32))) double pool[TileLds<T, DET>::kDoubles];
    const int L = logical_block();
    if (L >= nwork) return;
    const int2 w = work[L];
    // Descriptors copied up front, before any store of the kernel, so they
    // are fetched once as uniform (scalar) loads.
    const BufsD<T> B = dev_view(bufs[w.x]);
    const TopoD<T> tp = dev_view(topos[B.topo]);
    const int contact_full = P->contact_full;
    const InstState *s = B.s;
    const int phase = s->phase;
    if (s->model != LAW) return;   // served by the other law's launch
    if (phase == PH_CG || phase == PH_EVAL_HV) {
        tile_hessvec<T, LAW, DET>(tp, B, s, w.y, pool);
    } else if (phase == PH_GRAD || phase == PH_EVAL_GRAD || phase == PH_TRIAL) {
        const T alpha = phase == PH_TRIAL ? (T)s->alpha_ls : (T)0;
        tile_element<T, LAW, DET>(tp, B, s, w.y, alpha, contact_full, pool);
    }
}

// ---------------------------------------------------------------------------
// Newton init of one node block (phases GRAD, EVAL_GRAD after the element
// path of the same pass; INIT after an accepted line-search trial). Applies
// an accepted step u += alpha dx, gathers g and the node block from the tile
// and contact partials, forms the block (or scalar) Jacobi inverse, r = -g and
// z = M^-1 r on free nodes; partial sums of |g_free|^2 and r.z.
// Implicit steps (dt > 0): at the start of a time step (step_start) the
// velocity of the step just completed, v += (u - ut) / dt, and the new
// predictor ut = u + dt v are formed first; every init then adds the inertial
// gradient (m/dt^2)(u - ut), (m/dt^2) I to the node block, and the inertial
// energy (m/2dt^2)|u - ut|^2 to its own partial sum.
// ---------------------------------------------------------------------------
template <typename T, bool FRIC, int COH = kAlone>
__device__ __forceinline__ void node_init(const TopoD<T> &tp, const BufsD<T> &B, const InstState *s, int blk,
                                          bool apply, bool step_start, int block_jacobi) {
    const T alpha = (T)s->alpha_ls;
    const double dt = s->dt, mdt2 = s->mdt2;
    const bool dyn = dt > 0.0;
    double acc[3] = {0.0, 0.0, 0.0};   // |g_free|^2, r.z, inertial energy
    double unused = 0.0;
    const int i = blk * kBlock + threadIdx.x;
    if (i < tp.n) {
        T un[3] = {(T)0, (T)0, (T)0};
        if (apply || dyn) ld_vec<COH>(B.u, tp.n, i, un);
        if (apply) {
            T dd[3];
            ld_vec<COH>(B.dx, tp.n, i, dd);
#pragma unroll
            for (int d = 0; d < 3; d++) un[d] = fma_t(alpha, dd[d], un[d]);
            st_vec<COH>(B.u, tp.n, i, un);
            // contact nodes with friction also accumulate the increment in FP64
            if (FRIC && s->mu_f > 0.0) {
                const int jc = tp.cidx[i];
                if (jc >= 0) {
                    double fl[8];
                    ld_vec<COH>(B.fr, tp.nc, jc, fl);
#pragma unroll
                    for (int d = 0; d < 3; d++) fl[4 + d] += (double)alpha * (double)dd[d];
                    st_vec<COH>(B.fr, tp.nc, jc, fl);
                }
            }
        }
        T gsum[9];
#pragma unroll
        for (int c = 0; c < 9; c++) gsum[c] = (T)0;
        for (int q = tp.node_ent_off[i]; q < tp.node_ent_off[i + 1]; q++) {
            T src[9];
            ld_vec<COH>(B.pg, tp.nent, tp.node_ent[q], src);
#pragma unroll
            for (int c = 0; c < 9; c++) gsum[c] += src[c];
        }
        const int j = tp.cidx[i];
        if (j >= 0) {
            T src[9];
            ld_vec<COH>(B.cp, tp.nc, j, src);
#pragma unroll
            for (int c = 0; c < 9; c++) gsum[c] += src[c];
        }
        if (dyn && !tp.fixed[i]) {
            const T h = (T)dt;
            const T cm = (T)mdt2 * tp.nvol[i];
            double en = 0.0;
            T tv[3], vo[3] = {(T)0, (T)0, (T)0};
            ld_vec<COH>(B.ut, tp.n, i, tv);
            if (step_start) ld_vec<COH>(B.v, tp.n, i, vo);
#pragma unroll
            for (int d = 0; d < 3; d++) {
                const T ui = un[d];
                T ti = tv[d];
                if (step_start) {
                    const T vv = vo[d] + (ui - ti) / h;
                    B.v[3 * i + d] = vv;
                    ti = fma_t(h, vv, ui);
                    B.ut[3 * i + d] = ti;
                }
                const T w = ui - ti;
                gsum[d] = fma_t(cm, w, gsum[d]);
                en += (double)w * (double)w;
            }
            acc[2] = 0.5 * (double)cm * en;
            gsum[3] += cm;
            gsum[4] += cm;
            gsum[5] += cm;
        }
#pragma unroll
        for (int d = 0; d < 3; d++) B.g[3 * i + d] = gsum[d];
        T M[6] = {(T)0, (T)0, (T)0, (T)0, (T)0, (T)0};
        T rr[3] = {(T)0, (T)0, (T)0}, zz[3] = {(T)0, (T)0, (T)0};
        if (!tp.fixed[i]) {
            const T a = gsum[3], bb = gsum[4], c = gsum[5], d = gsum[6], e = gsum[7], f = gsum[8];
            const T m2 = a * bb - d * d;
            const T c00 = bb * c - f * f, c01 = e * f - d * c, c02 = d * f - bb * e;
            const T det = a * c00 + d * c01 + e * c02;
            if (block_jacobi && a > (T)0 && m2 > (T)0 && det > (T)0) {
                const T id = (T)1 / det;
                M[0] = c00 * id;
                M[1] = (a * c - e * e) * id;
                M[2] = m2 * id;
                M[3] = c01 * id;
                M[4] = c02 * id;
                M[5] = (d * e - a * f) * id;
            } else {
                M[0] = safe_recip(a);
                M[1] = safe_recip(bb);
                M[2] = safe_recip(c);
            }
#pragma unroll
            for (int d2 = 0; d2 < 3; d2++) rr[d2] = -gsum[d2];
            precond(M, rr, zz, true);
#pragma unroll
            for (int d2 = 0; d2 < 3; d2++) {
                acc[0] += (double)rr[d2] * (double)rr[d2];
                acc[1] += (double)rr[d2] * (double)zz[d2];
            }
        }
#pragma unroll
        for (int c = 0; c < 6; c++) B.dinv[6 * i + c] = M[c];
#pragma unroll
        for (int d = 0; d < 3; d++) B.r[3 * i + d] = rr[d];
        const T zero[3] = {(T)0, (T)0, (T)0};
        st_vec<COH>(B.z, tp.n, i, zz);
        st_vec<COH>(B.p, tp.n, i, zero);
        st_vec<COH>(B.dx, tp.n, i, zero);
    }
    block_reduce<3, false>(acc, unused);
    const int streams[3] = {RS_GG, RS_IRZ, RS_EN};
    store_partials<COH>(B.red, B.red_stride, streams, blk, acc);
}

// ---------------------------------------------------------------------------
// CG update of one node block (phases CG, EVAL_HV). Every block sums the tile
// pass's p.q partials (fixed order, so all blocks agree; block 0 records the
// sum for the finalize) and forms
// alpha = r.z / p.q; then it gathers q from the tile partials plus the contact
// block times p (read only where the element pass flagged the block nonzero)
// and, on free nodes, sets p = z + beta p_prev, dx += alpha p,
// r -= alpha q, z = M^-1 r, with partial sums of r.z and r.r. At p.q <= 0 CG
// stops (on its first iteration the preconditioned residual becomes the
// Newton direction). EVAL_HV writes q instead.
// ---------------------------------------------------------------------------
// One node's part of a CG update: request() asks for what depends on the node
// alone, gather() for its tile partials, form() completes q and p, apply()
// follows once alpha is known. Lanes past the last node repeat it.
template <typename T> struct NodeCg {
    int i, j;
    bool live;                     // a free node (free nodes are numbered first)
    int4 e4;
    int2 e2;
    T pp[3], zv[3], rv[3], dxv[3], M[6];
    T part[kGather][3];
    bool act;
    T pv[3], qv[3];

    template <int COH, bool EVAL>
    __device__ __forceinline__ void request(const TopoD<T> &tp, const BufsD<T> &B, int node) {
        i = min(node, tp.n - 1);
        live = node < (EVAL ? tp.n : tp.n_free);
        e4 = tp.node_ent4[i];
        e2 = tp.node_ent2[i];
        j = tp.cidx[i];
        ld_vec<COH>(B.p, tp.n, i, pp);
        if constexpr (EVAL) {
            ld_vec<COH>(B.z, tp.n, i, zv);
        } else {
            ld_vec<COH>(B.r, tp.n, i, rv);
            ld_vec<COH>(B.dx, tp.n, i, dxv);
            ld_vec<COH>(B.dinv, tp.n, i, M);
        }
    }

    // The node's tile partials: the first kGather entries come with the node,
    // their loads in flight together; an absent one (-1) reads nothing and
    // counts 0.
    template <int COH> __device__ __forceinline__ void gather(const TopoD<T> &tp, const BufsD<T> &B) {
        const int ent[kGather] = {e4.x, e4.y, e4.z, e4.w, e2.x, e2.y};
#pragma unroll
        for (int k = 0; k < kGather; k++) ld_vec_or0<COH>(B.pq, tp.nent, ent[k], part[k]);
        act = ld_flag_or0<COH>(B.cact, tp.nc, j);
    }

    template <bool DYN, int COH, bool EVAL>
    __device__ __forceinline__ void form(const TopoD<T> &tp, const BufsD<T> &B, const InstState *s, T beta, int cg_first) {
        if constexpr (!EVAL) precond(M, rv, zv, cg_first != 0);
#pragma unroll
        for (int d = 0; d < 3; d++) {
            pv[d] = fma_t(beta, pp[d], zv[d]);
            qv[d] = (T)0;
        }
        // summed in entry order; the rest from the node -> entry lists (1 % of
        // the nodes of the 50k fingertip)
#pragma unroll
        for (int k = 0; k < kGather; k++)
#pragma unroll
            for (int d = 0; d < 3; d++) qv[d] += part[k][d];
        if (e2.y >= 0)
            for (int q = tp.node_ent_off[i] + kGather; q < tp.node_ent_off[i + 1]; q++) {
                T v[3];
                ld_vec<COH>(B.pq, tp.nent, tp.node_ent[q], v);
#pragma unroll
                for (int d = 0; d < 3; d++) qv[d] += v[d];
            }
        if (act) {
            T c9[9];
            ld_vec<COH>(B.cp, tp.nc, j, c9);
            const T *H = c9 + 3;
            qv[0] += H[0] * pv[0] + H[3] * pv[1] + H[4] * pv[2];
            qv[1] += H[3] * pv[0] + H[1] * pv[1] + H[5] * pv[2];
            qv[2] += H[4] * pv[0] + H[5] * pv[1] + H[2] * pv[2];
        }
        if (DYN && s->mdt2 > 0.0 && i < tp.n_free) {
            const T cm = (T)s->mdt2 * tp.nvol[i];
#pragma unroll
            for (int d = 0; d < 3; d++) qv[d] = fma_t(cm, pv[d], qv[d]);
        }
    }

    // acc: r.z and r.r
    template <int COH>
    __device__ __forceinline__ void apply(const TopoD<T> &tp, const BufsD<T> &B, T alpha, bool negcurv, int cg_first,
                                          double (&acc)[2]) {
        if (!negcurv) {
            if (live) {
#pragma unroll
                for (int d = 0; d < 3; d++) {
                    dxv[d] = fma_t(alpha, pv[d], dxv[d]);
                    rv[d] = fma_t(-alpha, qv[d], rv[d]);
                    B.r[3 * i + d] = rv[d];
                }
                st_vec<COH>(B.p, tp.n, i, pv);
                st_vec<COH>(B.dx, tp.n, i, dxv);
                T zn[3];
                precond(M, rv, zn, false);
                st_vec<COH>(B.z, tp.n, i, zn);
                acc[0] += (double)rv[0] * (double)zn[0] + (double)rv[1] * (double)zn[1] + (double)rv[2] * (double)zn[2];
                acc[1] += (double)rv[0] * (double)rv[0] + (double)rv[1] * (double)rv[1] + (double)rv[2] * (double)rv[2];
            }
        } else if (cg_first && live) {
            st_vec<COH>(B.dx, tp.n, i, pv);
        }
    }
};

template <typename T, bool DYN, bool EVAL, int COH = kAlone>
__device__ __forceinline__ void node_update(const TopoD<T> &tp, const BufsD<T> &B, const InstState *s, int blk, int npq) {
    // solver scalars and this thread's node data first: their loads are in
    // flight while the block sums the p.q partials
    const double rz = uni<COH>(s->rz);
    const T beta = uni<COH>((T)s->beta);
    const int cg_first = uni<COH>((int)(s->cg_it == 0));
    double acc[2] = {0.0, 0.0};   // r.z, r.r
    NodeCg<T> c;
    c.template request<COH, EVAL>(tp, B, blk * kBlock + (int)threadIdx.x);
    c.template gather<COH>(tp, B);
    c.template form<DYN, COH, EVAL>(tp, B, s, beta, cg_first);
    const double pq = wave_sum_partials<COH>(B.red + RS_PQ * B.red_stride, npq);
    if (blk == 0 && threadIdx.x == 0) st_one<COH>((double *)(B.red + RS_PQN * B.red_stride), pq);
    if constexpr (EVAL) {
        if (c.live)
#pragma unroll
            for (int d = 0; d < 3; d++) B.qout[3 * c.i + d] = c.qv[d];
    } else {
        const bool negcurv = !(pq > 0.0);
        c.template apply<COH>(tp, B, negcurv ? (T)0 : (T)(rz / pq), negcurv, cg_first, acc);
    }
    // per-wavefront partials (kWaves per block), summed by the finalize
    acc[0] = wave_sum(acc[0]);
    acc[1] = wave_sum(acc[1]);
    if ((threadIdx.x & 63) == 0) {
        const int slot = kWaves * blk + (int)(threadIdx.x >> 6);
        st_one<COH>((double *)(B.red + RS_RZ * B.red_stride + slot), acc[0]);
        st_one<COH>((double *)(B.red + RS_RR * B.red_stride + slot), acc[1]);
    }
}

// Node blocks that a CG update works on: those with free nodes (numbered
// first); block 0 always, it records p.q.
__device__ __forceinline__ int cg_blocks(int n_free) { return n_free > kBlock ? (n_free + kBlock - 1) / kBlock : 1; }

// Line-search trial, node part: partial sums of g . dx (first trial of a
// line search) and, for implicit steps, of the inertial energy
// (m/2dt^2)|u + alpha dx - ut|^2 at the trial point.
template <typename T, int COH = kAlone>
__device__ __forceinline__ void node_trial(const TopoD<T> &tp, const BufsD<T> &B, const InstState *s, int blk) {
    double acc[2] = {0.0, 0.0};
    double unused = 0.0;
    const int i = blk * kBlock + threadIdx.x;
    if (i < tp.n) {
        T dd[3];
        ld_vec<COH>(B.dx, tp.n, i, dd);
        if (s->need_gd) {
            T gv[3];
            ld_vec<COH>(B.g, tp.n, i, gv);
#pragma unroll
            for (int d = 0; d < 3; d++) acc[0] += (double)gv[d] * (double)dd[d];
        }
        if (s->dt > 0.0 && !tp.fixed[i]) {
            const T alpha = (T)s->alpha_ls;
            T un[3], tv[3];
            ld_vec<COH>(B.u, tp.n, i, un);
            ld_vec<COH>(B.ut, tp.n, i, tv);
            double en = 0.0;
#pragma unroll
            for (int d = 0; d < 3; d++) {
                const T w = fma_t(alpha, dd[d], un[d]) - tv[d];
                en += (double)w * (double)w;
            }
            acc[1] = 0.5 * s->mdt2 * (double)tp.nvol[i] * en;
        }
    }
    block_reduce<2, false>(acc, unused);
    const int streams[2] = {RS_GD, RS_EN};
    store_partials<COH>(B.red, B.red_stride, streams, blk, acc);
}

// ---------------------------------------------------------------------------
// Node pass: one block per (instance, 256 nodes), after the tile pass of the
// same step. CG -> update; GRAD, EVAL_GRAD, INIT -> Newton init; TRIAL ->
// g . dx on the first trial of a line search and the inertial energy of
// implicit steps; other phases return.
// ---------------------------------------------------------------------------
// Friction lag data of the contact-eligible nodes of one node block.
template <typename T, int COH = kAlone>
__device__ __forceinline__ void node_lag(const TopoD<T> &tp, const BufsD<T> &B, const InstState *s, int blk) {
    const int i = blk * kBlock + threadIdx.x;
    if (i >= tp.n) return;
    const int j = tp.cidx[i];
    if (j < 0) return;
    double x[3], fl[8];
    T un[3];
    ld_vec<COH>(B.u, tp.n, i, un);
#pragma unroll
    for (int d = 0; d < 3; d++) x[d] = tp.X[3 * i + d] + (double)un[d];
    friction_lag(s, x, fl);
    st_vec<COH>(B.fr, tp.nc, j, fl);
}

// One node block of a job, whatever its phase. view(): the job's descriptors,
// asked for in each branch so that the team kernel holds only those in use.
// npq: partials of p.q (0: one per tile and contact block).
template <typename T, bool FRIC, int COH, class View>
__device__ __forceinline__ void node_block(View view, const InstState *s, int blk, int npq, int block_jacobi) {
    const int phase = uni<COH>((int)s->phase);
    if (phase == PH_EVAL_HV) {
        const auto V = view();
        node_update<T, true, true, COH>(V.tp, V.B, s, blk, npq ? npq : V.tp.ntile + V.tp.ncb);
    } else if (COH == kAlone && phase == PH_CG) {   // the team kernel's CG updates go through team_update
        const auto V = view();
        // a CG update changes free nodes only: blocks of fixed nodes (numbered
        // last) have nothing to do; block 0 always runs (it records p.q)
        if (blk > 0 && blk * kBlock >= V.tp.n_free) return;
        // the inertial term as a separate instance keeps it out of the
        // quasi-static CG update
        const int np = V.tp.ntile + V.tp.ncb;
        if (s->mdt2 > 0.0)
            node_update<T, true, false, COH>(V.tp, V.B, s, blk, np);
        else
            node_update<T, false, false, COH>(V.tp, V.B, s, blk, np);
    } else if (phase == PH_GRAD || phase == PH_EVAL_GRAD || phase == PH_INIT) {
        const auto V = view();
        node_init<T, FRIC, COH>(V.tp, V.B, s, blk, phase == PH_INIT && s->apply != 0, phase == PH_GRAD, block_jacobi);
    } else if (phase == PH_TRIAL && (s->need_gd || s->dt > 0.0)) {
        const auto V = view();
        node_trial<T, COH>(V.tp, V.B, s, blk);
    } else if (FRIC && phase == PH_LAG) {
        const auto V = view();
        node_lag<T, COH>(V.tp, V.B, s, blk);
    }
}

template <typename T> struct StepView {
    const TopoD<T> &tp;
    const BufsD<T> &B;
};

template <typename T, bool FRIC>
__global__ __launch_bounds__(kBlock) void k_node(const Topo<T> *topos, const InstBufs<T> *bufs, const int2 *work,
                                                 int nwork, const SolveParams *P) {
    const int L = logical_block();
    if (L >= nwork) return;
    const int2 w = work[L];
    // Descriptors copied up front, before any store of the kernel, so they
    // are fetched once as uniform (scalar) loads.
    const BufsD<T> B = dev_view(bufs[w.x]);
    const TopoD<T> tp = dev_view(topos[B.topo]);
    node_block<T, FRIC, kAlone>([&] { return StepView<T>{tp, B}; }, B.s, w.y, 0, P->block_jacobi);
}

// Newton test on |g_free| against the load step's first residual, then CG
// set-up with the inexact-Newton tolerance (finalising thread). Rounding
// floor: once the residual sits below floor_rtol * r0 and two accepted steps
// in a row whose predicted energy change lies within rounding have not halved
// the smallest residual of the step, the working precision cannot take it
// lower and the step ends with ST_FLOOR.
template <class StatePtr, class HistPtr>   // global-address-space pointers on the device
__device__ inline void newton_test(StatePtr s, HistPtr hist, const SolveParams *P, double gg, double rz) {
    s->gg = gg;
    const double gn = sqrt(gg);
    if (s->step_started) {
        s->r0 = gn;
        s->st_g0 = gn;
        s->step_started = 0;
        s->gbest = gn;
        s->stall = 0;
    } else if (s->apply) {
        // At the rounding floor the search direction is noise: accepted steps
        // do not reduce the residual, and the energy change they predict,
        // g.dx, lies within the energy's rounding noise. A step that predicts
        // a resolvable decrease means the iteration is still limited by
        // nonlinearity (stick-slip transitions of friction, large
        // rotations), so it does not count.
        const bool at_noise = fabs(s->gd) <= P->noise_eps * s->emag;
        if (gn <= 0.5 * s->gbest || !at_noise) {
            s->stall = 0;
        } else {
            s->stall++;
        }
        s->gbest = fmin(s->gbest, gn);
    }
    if (s->apply) {
        s->newton_it++;
        s->st_newton++;
        s->apply = 0;
    }
    if (gn <= fmax(P->newton_rtol * s->r0, P->newton_atol)) {
        end_step(s, hist, ST_OK);
    } else if (s->stall >= 2 && gn <= P->floor_rtol * s->r0) {
        end_step(s, hist, ST_FLOOR);
    } else if (s->newton_it >= P->max_newton) {
        end_step(s, hist, ST_NOT_CONVERGED);
    } else {
        // inexact Newton: forcing term (|g| / |g_start|)^p, p = 1/2 by default
        // (superlinear of order 1 + p, without tight solves late in a step)
        const double rel = gn / s->r0;
        const double eta = fmin(P->cg_eta_max, fmax(P->cg_rtol, P->eta_power == 1.0 ? rel : pow(rel, P->eta_power)));
        s->tol2 = eta * eta * gg;
        s->rz = rz;
        s->rr = gg;
        s->beta = 0.0;
        s->alpha = 0.0;
        s->cg_it = 0;
        s->phase = PH_CG;
    }
}

// End of a CG solve: the first line-search trial at alpha = 1 follows, with
// g . dx taken by its node pass.
__device__ inline void start_line_search(InstState *s) {
    s->last_cg = s->cg_it;
    s->alpha_ls = 1.0;
    s->halvings = 0;
    s->need_gd = 1;
    s->phase = PH_TRIAL;
}

// ---------------------------------------------------------------------------
// Finalize: one wavefront per live instance sums, in a fixed order, the
// partials its blocks wrote in this step's tile and node passes and takes the
// state-machine transition.
//   CG         alpha, beta, r.z; CG stop (tolerance, iteration cap, p.q <= 0)
//              -> TRIAL at alpha = 1.
//   GRAD       energy of the load step's start, then the Newton test.
//   TRIAL      Armijo test with the rounding floor noise_eps * sum of
//              energy-term magnitudes: accept -> INIT, else halve alpha or
//              end the load step.
//   INIT       Newton test.
//   EVAL_GRAD, EVAL_HV -> IDLE.
// ---------------------------------------------------------------------------
// W: in the team kernel the members of the team, each of which leaves one
// partial per wavefront of the CG sums.
template <typename T, int COH, class StatePtr>
__device__ __forceinline__ void finalize_wave(const TopoD<T> &tp, const BufsD<T> &B, StatePtr s, signed char *hist,
                                              const SolveParams *P, int W) {
    const int phase = s->phase;
    const int S = B.red_stride;
    const int nt = tp.ntile + tp.ncb, nn = (tp.n + kBlock - 1) / kBlock;
    if (phase == PH_LAG) {
        if ((threadIdx.x & 63) == 0) s->phase = s->after_lag;
        return;
    }
    if (phase == PH_CG || phase == PH_EVAL_HV) {
        const double pq = ld_one<COH>((const double *)(B.red + RS_PQN * S));   // the node pass's sum, as it applied it
        // the node pass's per-wavefront partials of its blocks with free nodes
        const int ncg = min(cg_blocks(tp.n_free), W);
        const double *const part[2] = {B.red + RS_RZ * S, B.red + RS_RR * S};
        double sums[2];
        wave_sums_partials<COH, 2>(part, kWaves * ncg, sums);
        const double rz = sums[0], rr = sums[1];
        if ((threadIdx.x & 63) != 0) return;
        s->pq = pq;
        if (phase == PH_EVAL_HV) {
            s->phase = PH_IDLE;
            return;
        }
        s->st_hv++;
        if (!(pq > 0.0)) {
            start_line_search(s);
            return;
        }
        s->alpha = s->rz / pq;
        s->cg_it++;
        s->st_cg++;
        s->beta = rz / s->rz;
        s->rz = rz;
        s->rr = rr;
        if (rr <= s->tol2 || s->cg_it >= P->max_cg) start_line_search(s);
    } else if (phase == PH_GRAD || phase == PH_EVAL_GRAD || phase == PH_TRIAL) {
        // tile partials, plus the nodes' inertial energy of implicit steps
        const double en = s->dt > 0.0 ? wave_sum_partials<COH>(B.red + RS_EN * S, nn) : 0.0;
        const double E = wave_sum_partials<COH>(B.red + RS_E * S, nt) + en;
        const double mag = wave_sum_partials<COH>(B.red + RS_MAG * S, nt) + en;
        const double mn = wave_min_partials<COH>(B.red + RS_MINJ * S, nt);
        double gg = 0.0, rz = 0.0, gd = 0.0;
        if (phase != PH_TRIAL) {
            gg = wave_sum_partials<COH>(B.red + RS_GG * S, nn);
            rz = wave_sum_partials<COH>(B.red + RS_IRZ * S, nn);
        } else if (s->need_gd) {
            gd = wave_sum_partials<COH>(B.red + RS_GD * S, nn);
        }
        if ((threadIdx.x & 63) != 0) return;
        const double Et = mn > 0.0 ? E : INFINITY;
        s->st_grad++;
        if (phase != PH_TRIAL) {
            s->E = Et;
            s->emag = mag;
            s->minJ = mn;
            s->apply = 0;
            if (phase == PH_EVAL_GRAD) {
                s->gg = gg;
                s->phase = PH_IDLE;
            } else {
                newton_test(s, hist, P, gg, rz);
            }
            return;
        }
        if (s->need_gd) {
            s->gd = gd;
            s->need_gd = 0;
        }
        s->st_ls++;
        const double noise = P->noise_eps * s->emag;
        if (mn > 0.0 && Et <= s->E + P->c1 * s->alpha_ls * s->gd + noise) {
            s->E = Et;
            s->emag = mag;
            s->minJ = mn;
            s->apply = 1;
            s->phase = PH_INIT;
        } else if (s->halvings >= P->max_halvings) {
            end_step(s, hist, mn > 0.0 ? ST_NOT_CONVERGED : ST_INVERSION);
        } else {
            s->halvings++;
            s->alpha_ls *= 0.5;
        }
    } else if (phase == PH_INIT) {
        const double gg = wave_sum_partials<COH>(B.red + RS_GG * S, nn);
        const double rz = wave_sum_partials<COH>(B.red + RS_IRZ * S, nn);
        if ((threadIdx.x & 63) != 0) return;
        newton_test(s, hist, P, gg, rz);
    }
}

template <typename T>
__global__ __launch_bounds__(64) void k_finalize(const Topo<T> *topos, const InstBufs<T> *bufs, const int *live,
                                                 int nlive, const SolveParams *P) {
    if ((int)blockIdx.x >= nlive) return;
    const BufsD<T> B = dev_view(bufs[live[blockIdx.x]]);
    const TopoD<T> tp = dev_view(topos[B.topo]);
    finalize_wave<T, kAlone>(tp, B, B.s, (signed char *)B.hist, P, 0x7fffffff);   // B.s: global-address-space pointer on the device
}

// ---------------------------------------------------------------------------
// Persistent team kernel: all solver steps of a job in one launch.
//
// A team is W workgroups, on one XCD or (few jobs on large meshes) on several,
// that advance one job after another: tile
// pass, team barrier, node pass, team barrier, and the finalize, which every
// member takes for itself from the same partials in the same order on its own
// LDS copy of the job's state, so all members take the same transition. Teams
// are independent of each other: one team's node pass (bound by memory)
// overlaps another's tile pass (bound by vector arithmetic), no job waits for
// another's slower pass, and a step of a small job costs two barriers instead
// of three kernel boundaries.
//
// Members of one XCD share its L2, so nothing has to be written back or
// invalidated at a barrier: an agent-scope fence costs 59 ns per workgroup and
// barrier, one after another on an XCD (measured; 32 workgroups: 2.8 us).
// Stores are complete in the L2 once vmcnt is 0, and everything a team-mate
// may have written is loaded past the CU's vector cache (ld_vec, ld_one).
// Over several XCDs the stores go through to memory as well (kChip): 2.0 us
// for a barrier with stores before and loads after it, 0.65 us on one XCD.
// A workgroup reads the XCD it runs on from the hardware and is a member of a
// team there, so a team is where its kind needs it however workgroups were
// dealt; members that don't come make their team give up at its first meeting,
// below.
//
// Every wait ends. A team first meets: its members are counted in, and a
// member that has waited kMeetTicks for the rest calls the team off, once and
// for all, by a bit in the counter that only an incomplete team can get; no
// job state has been touched by then and the host runs those jobs through the
// other kernels. Teams that gather after that in the same launch, in the
// places of others that left, hardly wait again. A team that has met is resident as a whole, runs the same
// sequence of barriers in every member, and is never waited for by another
// team. A barrier that should not come about for kStuckTicks all the same
// ends the launch and is reported.
// ---------------------------------------------------------------------------
struct TeamDesc {
    int job_off, job_n;         // its jobs in the list
};
// One place of the plan: an XCD, or several consecutive ones that its teams span.
struct XcdDesc {
    int team0, nteam, W, pad;   // teams team0 .. team0 + nteam - 1 of W workgroups each
};
// The launch's XCDs among the device's `count`: places begin at XCD `first` and
// are 1 << shift XCDs each.
struct XcdMap {
    int first, count, shift;
};
// Arrivals are counted in groups of kTeamGroup members, the last of a group
// arriving for it at the team's counter: arrivals at one address are served
// one after another (28 ns each).
constexpr int kTeamGroup = 16, kTeamGroups = 16;
struct alignas(128) TeamLine {
    unsigned v;
    char pad[124];
};
struct TeamSync {
    TeamLine flag;                  // 2 * (last complete barrier) + stop, or kCalledOff
    TeamLine top;                   // arrivals of groups, and the stop request
    TeamLine group[kTeamGroups];    // arrivals of members
    unsigned member[kTeamGroup * kTeamGroups];   // the last launch in which a workgroup was this member
};
constexpr int kMaxXcds = 16;
// done, calledoff and stuck only grow, and the host takes differences between
// launches, which hold when they wrap; over (a team has seen that the launch is
// to end), gone (a team has been called off) and steps, a maximum over the
// teams, are the launch's own: the last workgroup to leave clears them.
struct alignas(8) TeamStat {
    unsigned done, over;   // read together
    unsigned calledoff, stuck, steps, gone;
};
// Pinned: the kernel's counters as of its last launch, and the host's wish that
// the launch in flight ends.
struct TeamHost {
    TeamStat stat;
    unsigned yield;
};
struct TeamCtl {
    TeamLine ticket[kMaxXcds];   // kChip: memberships taken, per place of the plan
    TeamLine leave;              // workgroups that have left
    // the host's mirror of the states, and its words (pinned); here, not in
    // the arguments, which would hold scalar registers throughout
    InstState *mirror;
    TeamHost *host;
    TeamSync sync[1];            // one per team
};
constexpr unsigned kCalledOff = 0xffffffffu;
constexpr unsigned kCalledOffBit = 0x80000000u;
constexpr unsigned kStopUnit = 1u << 24;                    // in the top counter, above any count of arrivals
constexpr unsigned kArrivals = kStopUnit - 1;
// 20 ms of the 100 MHz clock: on a free device the workgroups of a launch are
// all there within tens of microseconds, behind another kernel's last blocks
// within that kernel's tail.
constexpr unsigned long long kMeetTicks = 2000000ull;
constexpr unsigned long long kStuckTicks = 2000000000ull;   // 20 s
// A launch to the end holds its XCDs for 20 ms at most, since other streams'
// kernels wait for it. Every kTeamPoll solver steps (2.4 ms of the largest
// batch) a team looks at the clock, and every millisecond at the host's wish, a
// read over the bus; the first to see an end tells the others.
constexpr unsigned long long kLaunchTicks = 2000000ull, kLookTicks = 100000ull;
constexpr int kTeamPoll = 16;
enum : int { kStopDone = 1, kStopPoll = 2 };                // reasons to end early: see k_team

template <class U> __device__ __forceinline__ U ag_load(const U *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class U> __device__ __forceinline__ void ag_store(U *p, U v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class U> __device__ __forceinline__ U ag_add(U *p, U v) {
    return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Entry i of a table that the launch does not change, by scalar loads.
template <class S, class P> __device__ __forceinline__ S ld_table(const P *p, int i) {
    static_assert(sizeof(S) == sizeof(P) && sizeof(S) % 8 == 0, "table entry");
    const auto q = (const __attribute__((address_space(4))) unsigned long long *)(p + i);
    unsigned long long w[sizeof(S) / 8];
#pragma unroll
    for (int k = 0; k < (int)(sizeof(S) / 8); k++) w[k] = q[k];
    S out;
    __builtin_memcpy(&out, w, sizeof out);
    return out;
}

// The descriptors of job `job`, fetched anew at each use: held over a whole
// step they would take 100 scalar registers, which spill.
template <typename T> struct JobView {
    BufsD<T> B;
    TopoD<T> tp;
    __device__ __forceinline__ JobView(const Topo<T> *topos, const InstBufs<T> *bufs, int job) {
        asm volatile("" : "+s"(job));
        B = ld_table<BufsD<T>>(bufs, job);
        tp = ld_table<TopoD<T>>(topos, B.topo);
    }
};

// Member `rank`'s group among the W members: up to kTeamGroup members arrive
// at the top counter themselves.
struct TeamGroup {
    unsigned index, many, size, many_top;   // its group, groups, members of its group, arrivals at the top
    __device__ __forceinline__ TeamGroup(unsigned W, unsigned rank) {
        index = rank / kTeamGroup;
        many = (W + kTeamGroup - 1) / kTeamGroup;
        size = index + 1 < many ? kTeamGroup : W - index * kTeamGroup;
        many_top = many > 1 ? many : W;
    }
};

// Barrier number `ph` of a team (the meeting is number 1), in two halves so
// that loads which do not depend on it can go out in between. Member `rank`'s
// thread 0 arrives once its workgroup's stores are in the L2. A stop request
// of member 0 is passed on to all members with the flag.
__device__ __forceinline__ void team_arrive(TeamSync *ts, unsigned ph, unsigned W, unsigned rank, bool stop) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wavefront's stores are in the L2
    __syncthreads();
    if (threadIdx.x == 0) {
        const TeamGroup g(W, rank);
        bool last = true;
        if (g.many > 1) last = ag_add(&ts->group[g.index].v, 1u) + 1 == ph * g.size;
        if (stop) ag_add(&ts->top.v, kStopUnit);
        if (last) {
            const unsigned now = ag_add(&ts->top.v, 1u) + 1;
            if ((now & kArrivals) == ph * g.many_top) ag_store(&ts->flag.v, 2 * ph + (now >= kStopUnit ? 1u : 0u));
        }
    }
}

// Whether a launch to the end is over, looked up by a thread of member 0 while
// thread 0 waits at the second barrier of a step, where no loads are in flight
// whose waits a branch would make strict (at the first, behind the node pass's
// requests, it cost 0.5 of 11.7 us a step). Its request is in the L2 before
// member 0 arrives at the first barrier of the next step, whose flag tells all
// members. In LDS: arguments kept in scalar registers throughout would be
// spilled.
struct TeamLook {
    unsigned long long end, next;   // when the launch is over, and when to look again
    TeamStat *stat;
    const unsigned *yield;
    int on;
    unsigned launch;
    __device__ __forceinline__ void look_up(TeamSync *ts, int c) {
        if (threadIdx.x != kBlock - 64 || on == 0 || c % kTeamPoll != kTeamPoll - 1) return;
        const unsigned long long now = wall_clock64();
        if (now < next) return;
        next = now + kLookTicks;
        if (now < end && __hip_atomic_load(yield, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) == 0) return;
        ag_store(&stat->over, 1u);
        ag_add(&ts->top.v, kStopUnit);
        // both arrive before this workgroup can leave: the last one clears them
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
};

// Returns 0, 1 (stop) or -1 (the barrier did not come about).
__device__ __forceinline__ int team_wait(TeamSync *ts, unsigned ph, int *sh, TeamStat *stat) {
    if (threadIdx.x == 0) {
        unsigned long long t0 = 0;
        unsigned v;
        for (unsigned n = 1; (v = ag_load(&ts->flag.v)) < 2 * ph; n++) {
            __builtin_amdgcn_s_sleep(1);
            if ((n & 0xfff) == 0) {
                const unsigned long long now = wall_clock64();
                if (t0 == 0) {
                    t0 = now;
                } else if (now - t0 > kStuckTicks) {
                    ag_add(&stat->stuck, 1u);
                    ag_store(&ts->flag.v, kCalledOff);
                }
            }
        }
        sh[0] = v == kCalledOff ? -1 : (int)(v & 1u);
    }
    __syncthreads();
    const int r = __builtin_amdgcn_readfirstlane(sh[0]);
    asm volatile("" ::: "memory");
    return r;
}

// First meeting of a team (thread 0 of each member): true once all W members
// are there. It leaves the counters as after barrier 1.
__device__ __forceinline__ bool team_meet(TeamSync *ts, unsigned W, unsigned rank, TeamStat *stat) {
    const TeamGroup g(W, rank);
    bool last = true;
    if (g.many > 1) last = ag_add(&ts->group[g.index].v, 1u) + 1 == g.size;
    if (last) {
        const unsigned now = ag_add(&ts->top.v, 1u) + 1;
        if (now & kCalledOffBit) return false;
        if (now == g.many_top) {
            ag_store(&ts->flag.v, 2u);
            return true;
        }
    }
    const unsigned long long t0 = wall_clock64();
    for (;;) {
        const unsigned v = ag_load(&ts->flag.v);
        if (v == kCalledOff) return false;
        if (v >= 2u) return true;
        __builtin_amdgcn_s_sleep(8);
        const unsigned long long waited = wall_clock64() - t0;
        if (waited > kMeetTicks || (waited > kMeetTicks / 100 && ag_load(&stat->gone) != 0)) {
            unsigned a = ag_load(&ts->top.v);
            while (a < g.many_top) {   // incomplete and not called off
                if (__hip_atomic_compare_exchange_strong(&ts->top.v, &a, a | kCalledOffBit, __ATOMIC_RELAXED,
                                                         __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                    ag_add(&stat->calledoff, 1u);
                    ag_store(&stat->gone, 1u);
                    ag_store(&ts->flag.v, kCalledOff);
                    return false;
                }
            }
            // complete, or called off by another member: the flag follows
        }
    }
}

// Word i of a table that the launch does not change, by a scalar load.
__device__ __forceinline__ int ld_int(const int *p, int i) {
    return ((const __attribute__((address_space(4))) int *)p)[i];
}

// Entries and tets of one tile.
template <typename T> struct TileSpan {
    int e0, ne, k0, nk;
    __device__ __forceinline__ TileSpan(const TopoD<T> &tp, int t) {
        e0 = ld_int((const int *)tp.tile_ent, t);
        ne = ld_int((const int *)tp.tile_ent, t + 1) - e0;
        k0 = ld_int((const int *)tp.tile_tet, t);
        nk = ld_int((const int *)tp.tile_tet, t + 1) - k0;
    }
};

// Hessian-vector pass of one team member: tile blocks rank, rank + W, ... of
// its job, then contact blocks. The arithmetic is tile_hessvec's. A member
// walks several tiles (20 for a job of the 50k fingertip among 256) and would
// wait for memory three times in each: everything the next tile needs is
// therefore requested while the current one's tets are computed, its node
// vectors behind the first and second tet, each tet record behind the other
// tet. These requests are unconditional (past the last tile they repeat it),
// since the compiler's wait after a branch counts as if none had been made
// and would wait for them too. The LDS sums alternate between two halves, so
// two block barriers per tile are enough, and p.q is summed over all of the
// member's blocks before it is reduced and stored as one partial.
template <typename T, int LAW, int COH>
__device__ __forceinline__ void team_hessvec(const TopoD<T> &tp, const BufsD<T> &B, const InstState *s, int rank, int W,
                                             double *pool) {
    static_assert(kTileTets == 2 * kBlock, "two tets per thread");
    // A team may be larger than this mesh's list (jobs on larger meshes share
    // it): a member without an item has no slot among the partials, whose
    // stride is the mesh's.
    if (rank >= tp.ntile + tp.ncb) return;
    const T beta = uni<COH>((T)s->beta);
    const T mu = uni<COH>((T)s->mu), lam = uni<COH>((T)s->lam);
    const double cm = uni<COH>(s->mdt2);
    T *su = (T *)(pool + 6 * kTileNodes), *sp = su + kSw * kTileNodes;
    const int tid = threadIdx.x;
    double pq = 0.0;
    if (rank < tp.ntile) {
        int half = 0;
        TileSpan<T> cur(tp, rank);
        int gid = tp.ent_node[cur.e0 + min(tid, cur.ne - 1)], sl = tp.ent_slot[cur.e0 + min(tid, cur.ne - 1)];
        TetWords<T> r0, r1;
        fetch_tet(tp, cur.k0 + min(tid, cur.nk - 1), r0);
        T uv[3], pp[3], zv[3];
        ld_vec<COH>(B.u, tp.n, gid, uv);
        ld_vec<COH>(B.p, tp.n, gid, pp);
        ld_vec<COH>(B.z, tp.n, gid, zv);
        fetch_tet(tp, cur.k0 + min(tid + kBlock, cur.nk - 1), r1);
        for (int t = rank;;) {
            double *sa = pool + half;
            const int tn = t + W;
            const bool more = tn < tp.ntile;
            const TileSpan<T> nxt(tp, more ? tn : t);
            const int en = nxt.e0 + min(tid, nxt.ne - 1);
            const int gidn = tp.ent_node[en], sln = tp.ent_slot[en];
            if (tid < cur.ne) {
                T pv[3];
#pragma unroll
                for (int d = 0; d < 3; d++) {
                    pv[d] = fma_t(beta, pp[d], zv[d]);
                    su[kSw * sl + d] = uv[d];
                    sp[kSw * sl + d] = pv[d];
                    sa[3 * sl + d] = 0.0;
                }
                if (cm > 0.0 && tp.owner[cur.e0 + tid])
                    pq += cm * (double)tp.nvol[gid] *
                          ((double)pv[0] * (double)pv[0] + (double)pv[1] * (double)pv[1] + (double)pv[2] * (double)pv[2]);
            }
            __syncthreads();
            ld_vec<COH>(B.u, tp.n, gidn, uv);
            ld_vec<COH>(B.p, tp.n, gidn, pp);
            ld_vec<COH>(B.z, tp.n, gidn, zv);
            auto tet = [&](const TetWords<T> &rec) {
                int l[4];
                T f[4][3], wp[4][3], e_pq = (T)0;
                if (!tet_hessvec<T, LAW>(rec, su, sp, mu, lam, l, f, wp)) return;
#pragma unroll
                for (int a = 0; a < 4; a++) {
#pragma unroll
                    for (int d = 0; d < 3; d++) atomicAdd(sa + 3 * l[a] + d, (double)f[a][d]);
                    e_pq += wp[a][0] * f[a][0] + wp[a][1] * f[a][1] + wp[a][2] * f[a][2];
                }
                pq += (double)e_pq;
            };
            if (tid < cur.nk) tet(r0);
            fetch_tet(tp, nxt.k0 + min(tid, nxt.nk - 1), r0);
            if (tid + kBlock < cur.nk) tet(r1);
            fetch_tet(tp, nxt.k0 + min(tid + kBlock, nxt.nk - 1), r1);
            __syncthreads();
            if (tid < cur.ne) {
                T out[3];
#pragma unroll
                for (int d = 0; d < 3; d++) out[d] = (T)sa[3 * sl + d];
                st_vec<COH>(B.pq, tp.nent, cur.e0 + tid, out);
            }
            if (!more) break;
            half = 3 * kTileNodes - half;
            t = tn;
            cur = nxt;
            gid = gidn;
            sl = sln;
        }
    }
    // contact blocks follow the tiles in the members' turn
    int i0 = rank;
    if (i0 < tp.ntile) i0 += (tp.ntile - i0 + W - 1) / W * W;
    for (int i = i0; i < tp.ntile + tp.ncb; i += W) pq += contact_hessvec<T, COH>(tp, B, (i - tp.ntile) * kBlock + tid, beta);
    double acc[1] = {pq}, unused = 0.0;
    block_reduce<1, false>(acc, unused);
    const int streams[1] = {RS_PQ};
    store_partials<COH>(B.red, B.red_stride, streams, rank, acc);
}

// CG update of one team member: node blocks rank, rank + W, ... with p.q
// formed once and the sums of r.z and r.r taken over all of them. c: the first
// block, requested before the barrier: its r, dx, p and M^-1 are this thread's
// own, the lists the mesh's. A small team's step is a chain of latencies, and
// this takes one out: load steps of the 3072-tet block 14.5 -> 13.7 ms (FP64),
// 5k tets 1.56 -> 1.48 ms (FP32), 50k 12.0 -> 11.4 ms (FP64); members of batches
// with several blocks each neither gain nor lose. The same for the tile pass's
// first records would hold them over the finalize: 161 registers for 106 and
// 5 to 13 % on FP32 batches.
template <typename T, int COH>
__device__ __forceinline__ void team_update(const TopoD<T> &tp, const BufsD<T> &B, const InstState *s, int rank, int W,
                                            NodeCg<T> &c) {
    const double rz = uni<COH>(s->rz);
    const T beta = uni<COH>((T)s->beta);
    const int cg_first = uni<COH>((int)(s->cg_it == 0));
    const int nb = cg_blocks(tp.n_free);
    if (rank >= nb) return;
    double acc[2] = {0.0, 0.0};
    const double *const part[1] = {B.red + RS_PQ * B.red_stride};
    double sum[1];
    wave_sums_partials<COH, 1>(part, min(W, tp.ntile + tp.ncb), sum);
    const double pq = uni<COH>(sum[0]);
    const bool negcurv = !(pq > 0.0);
    const T alpha = negcurv ? (T)0 : (T)(rz / pq);
    for (int blk = rank;;) {
        // the next block's node data are requested behind this block's gather
        const bool more = blk + W < nb;
        c.template gather<COH>(tp, B);
        NodeCg<T> n;
        n.template request<COH, false>(tp, B, (more ? blk + W : blk) * kBlock + (int)threadIdx.x);
        c.template form<true, COH, false>(tp, B, s, beta, cg_first);
        c.template apply<COH>(tp, B, alpha, negcurv, cg_first, acc);
        if (!more) break;
        blk += W;
        c = n;
    }
    if (rank == 0 && threadIdx.x == 0) st_one<COH>((double *)(B.red + RS_PQN * B.red_stride), pq);
    acc[0] = wave_sum(acc[0]);
    acc[1] = wave_sum(acc[1]);
    if ((threadIdx.x & 63) == 0) {
        const int slot = kWaves * rank + (int)(threadIdx.x >> 6);
        st_one<COH>((double *)(B.red + RS_RZ * B.red_stride + slot), acc[0]);
        st_one<COH>((double *)(B.red + RS_RR * B.red_stride + slot), acc[1]);
    }
}

__device__ __forceinline__ bool running_phase(int ph) { return ph != PH_IDLE && ph != PH_DONE; }

// LAWS: constitutive laws among the jobs (1 Neo-Hookean, 2 co-rotational, 3
// both). COH: kXcd, or kChip with teams over several XCDs each. stop_on: with
// kStopDone the launch ends once `done` has reached stop_at or a team has said
// so, with kStopPoll after kLaunchTicks or at the host's wish; otherwise each
// job takes `steps` solver steps or ends.
// At least 4 (FP32) and 2 (FP64) wavefronts per SIMD, as many as it needs
// registers for; teams are as large as fit at once.
template <typename T, int LAWS, int COH>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 2))) void k_team(const Topo<T> *topos, const InstBufs<T> *bufs, const int *jobs,
                                                 const TeamDesc *teams, const XcdDesc *xcds, TeamCtl *ctl,
                                                 TeamStat *stat, const SolveParams *P, XcdMap map, int steps, int stop_on,
                                                 unsigned stop_at, unsigned launch) {
    using Lds = TileLds<T, false>;
    __shared__ __attribute__((aligned(32))) double pool[Lds::kDoubles > Lds::kTeamHv ? Lds::kDoubles : Lds::kTeamHv];
    __shared__ InstState S;
    __shared__ int sh[1];
    __shared__ TeamLook L;
    static_assert(sizeof(InstState) % 8 == 0, "copied as 8-byte words");
    constexpr int kStateWords = sizeof(InstState) / 8;
    // hardware register 20: XCC_ID, low four bits
    const int xcd = __builtin_amdgcn_readfirstlane((int)(__builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15u));
    const int at = (xcd >= map.first ? xcd - map.first : xcd - map.first + map.count) >> map.shift;
    const XcdDesc X = ld_table<XcdDesc>(xcds, at);
    // Workgroups are dealt to the XCDs, and on each to its CUs, in turn, so
    // consecutive rows of the grid are consecutive CUs, and a team on one XCD
    // stands on as many as it has members. By the order in which workgroups came
    // to a counter, teams of 21 stood on 8 to 21 of the 32, by what else the
    // kernel does before it counts (48 jobs on three fingertips: 11.8 to 12.4 ms,
    // by rows 11.6; 256 jobs on the 50k one 127 -> 121 ms). Were they ever dealt
    // otherwise, a member would be there twice: it gives up the second time, and
    // the team that lacks another does not meet. Teams over several XCDs take
    // members as they come: by rows the FP64 step of the 50k fingertip took 2.5 %
    // more, and with the rows of one XCD after those of another three FP32 jobs 3 %
    // more (their node blocks, fewer than the members, on half of the XCDs).
    int place = (int)blockIdx.y;
    if (threadIdx.x == 0) {
        if constexpr (COH == kChip) place = (int)ag_add(&ctl->ticket[at].v, 1u);
        TeamSync *ts = &ctl->sync[X.team0 + place / X.W];
        if (place >= X.nteam * X.W ||
            (COH != kChip && __hip_atomic_exchange(&ts->member[place % X.W], launch, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT) == launch) ||
            !team_meet(ts, (unsigned)X.W, (unsigned)(place % X.W), stat))
            place = -1;
        sh[0] = place;
        const unsigned long long now = wall_clock64();
        L = {now + kLaunchTicks, now + kLookTicks, stat, &ctl->host->yield, stop_on & kStopPoll, launch};
    }
    __syncthreads();
    place = __builtin_amdgcn_readfirstlane(sh[0]);
    if (place >= 0) {
        const int team = X.team0 + place / X.W, rank = place % X.W, W = X.W;
        const TeamDesc D = ld_table<TeamDesc>(teams, team);
        TeamSync *ts = &ctl->sync[team];
        unsigned ph = 1;
        int most = 0, r = 0;
        for (int q = 0; q < D.job_n && r >= 0; q++) {
            const int job = ld_int(jobs, D.job_off + q);
            // The state as the host or the last launch left it; member 0
            // writes it back at the end.
            unsigned long long *ls = (unsigned long long *)&S;
            int nnb, blocks;   // node blocks; tile and contact blocks
            __syncthreads();
            {
                const JobView<T> V(topos, bufs, job);
                nnb = (V.tp.n + kBlock - 1) / kBlock;
                blocks = V.tp.ntile + V.tp.ncb;
                const unsigned long long *gs = (const unsigned long long *)(InstState *)V.B.s;
                for (int k = threadIdx.x; k < kStateWords; k += kBlock) ls[k] = gs[k];
            }
            __syncthreads();
            const bool nh = LAWS == 1 || (LAWS == 3 && uni<kXcd>((int)S.model) == LAW_NH);
            int c = 0, phase = uni<kXcd>((int)S.phase);
            bool stop = false;
            for (; c < steps && running_phase(phase) && !stop; c++) {
                bool ask = false;
                if ((stop_on & kStopDone) && rank == 0 && threadIdx.x == 0) {
                    const unsigned long long both = ag_load((const unsigned long long *)&stat->done);
                    ask = (int)((unsigned)both - stop_at) >= 0 || (both >> 32) != 0;
                }
                if (phase == PH_CG || phase == PH_EVAL_HV) {
                    const JobView<T> V(topos, bufs, job);
                    if ((LAWS & 1) && nh)
                        team_hessvec<T, LAW_NH, COH>(V.tp, V.B, &S, rank, W, pool);
                    else if (LAWS & 2)
                        team_hessvec<T, LAW_CR, COH>(V.tp, V.B, &S, rank, W, pool);
                } else if (phase == PH_GRAD || phase == PH_EVAL_GRAD || phase == PH_TRIAL) {
                    const T alpha = phase == PH_TRIAL ? uni<kXcd>((T)S.alpha_ls) : (T)0;
                    const JobView<T> V(topos, bufs, job);
                    const int ntb = V.tp.ntile + V.tp.ncb;
                    for (int i = rank; i < ntb; i += W) {
                        if ((LAWS & 1) && nh)
                            tile_element<T, LAW_NH, false, COH>(V.tp, V.B, &S, i, alpha, P->contact_full, pool);
                        else if (LAWS & 2)
                            tile_element<T, LAW_CR, false, COH>(V.tp, V.B, &S, i, alpha, P->contact_full, pool);
                    }
                }
                team_arrive(ts, ++ph, W, rank, ask);
                if (phase == PH_CG) {
                    const JobView<T> V(topos, bufs, job);
                    NodeCg<T> first;
                    first.template request<COH, false>(V.tp, V.B, rank * kBlock + (int)threadIdx.x);
                    r = team_wait(ts, ph, sh, stat);
                    if (r < 0) break;
                    stop = r > 0;
                    team_update<T, COH>(V.tp, V.B, &S, rank, W, first);
                } else {
                    r = team_wait(ts, ph, sh, stat);
                    if (r < 0) break;
                    stop = r > 0;
                    for (int i = rank; i < nnb; i += W)
                        node_block<T, true, COH>([&] { return JobView<T>(topos, bufs, job); }, &S, i, min(W, blocks),
                                                 P->block_jacobi);
                }
                team_arrive(ts, ++ph, W, rank, false);
                if (rank == 0) L.look_up(ts, c);
                r = team_wait(ts, ph, sh, stat);
                if (r < 0) break;
                if (threadIdx.x < 64) {
                    const JobView<T> V(topos, bufs, job);
                    finalize_wave<T, COH>(V.tp, V.B, &S, rank == 0 ? (signed char *)V.B.hist : nullptr, P, W);
                }
                __syncthreads();
                const int next = uni<kXcd>((int)S.phase);
                // A tile pass right after a trial or gradient would overwrite
                // the energy partials that slower members still sum.
                if ((phase == PH_TRIAL || phase == PH_GRAD) && (next == PH_TRIAL || next == PH_GRAD)) {
                    team_arrive(ts, ++ph, W, rank, false);
                    r = team_wait(ts, ph, sh, stat);
                    if (r < 0) break;
                }
                phase = next;
            }
            most = max(most, c);
            if (rank == 0 && r >= 0) {
                if (threadIdx.x == 0) {
                    if (c > 0 && !running_phase(phase)) ag_add(&stat->done, 1u);
                    S.launch = L.launch;
                }
                __syncthreads();
                const JobView<T> V(topos, bufs, job);
                unsigned long long *gs = (unsigned long long *)(InstState *)V.B.s;
                unsigned long long *hs = (unsigned long long *)(ctl->mirror + job);
                for (int k = threadIdx.x; k < kStateWords; k += kBlock) gs[k] = hs[k] = ls[k];
            }
        }
        if (rank == 0 && threadIdx.x == 0)
            __hip_atomic_fetch_max(&stat->steps, (unsigned)most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // the last workgroup to leave hands the launch's counters to the host
    // (this thread's own additions to them have arrived before it leaves) and
    // clears the teams' for the next launch
    if (threadIdx.x == 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (threadIdx.x == 0 && ag_add(&ctl->leave.v, 1u) == gridDim.x * gridDim.y - 1) {
        TeamStat *stat_mirror = &ctl->host->stat;
        stat_mirror->done = ag_load(&stat->done);
        stat_mirror->calledoff = ag_load(&stat->calledoff);
        stat_mirror->stuck = ag_load(&stat->stuck);
        stat_mirror->steps = ag_load(&stat->steps);
        ag_store(&stat->steps, 0u);
        ag_store(&stat->gone, 0u);
        ag_store(&stat->over, 0u);
        for (int x = 0; x < kMaxXcds; x++) {
            const XcdDesc Y = ld_table<XcdDesc>(xcds, x);
            for (int t = Y.team0; t < Y.team0 + Y.nteam; t++) {
                ag_store(&ctl->sync[t].flag.v, 0u);
                ag_store(&ctl->sync[t].top.v, 0u);
                for (int g = 0; kTeamGroup * g < Y.W; g++) ag_store(&ctl->sync[t].group[g].v, 0u);
            }
            if (COH == kChip) ag_store(&ctl->ticket[x].v, 0u);
        }
        ag_store(&ctl->leave.v, 0u);
    }
}

// XCD of each workgroup of a small launch (set-up probe: how workgroups are
// dealt to the XCDs).
__global__ void k_xcds(unsigned *out) {
    if (threadIdx.x == 0) out[blockIdx.x] = __builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15u;
}

// ---------------------------------------------------------------------------
// Contact patch of one instance at its current state, written straight to
// pinned host memory (no copies after the kernel): one thread per eligible
// node, each block compacting its nodes that carry a contact force, phi < 0 or
// friction from the lag state, into its own segment of the lists (in eligible
// order): ids, forces on the skin -k min(0, phi) n minus the friction
// gradient, phi; and its count and FP64 resultant into its head. With lists =
// false only the heads. The signed distance takes some hundred FP64
// instructions a node, so the nodes are spread over as many CUs as there are
// blocks. A call for the count and resultant of 3757 nodes took 47 us when one
// block walked them and two copies followed; it takes 17 us, 4 of them the kernel.
// ---------------------------------------------------------------------------
struct PatchHead {
    double F[3];
    int count, pad;
};

template <typename T>
__global__ __launch_bounds__(kBlock) void k_contact_patch(const Topo<T> *topos, const InstBufs<T> *bufs, int inst,
                                                          PatchHead *heads, int *ids, double *f, double *phi_out,
                                                          bool lists) {
    __shared__ int wave_cnt[kWaves];
    __shared__ double wave_f[kWaves][3];
    const BufsD<T> B = dev_view(bufs[inst]);
    const TopoD<T> tp = dev_view(topos[B.topo]);
    const InstState *s = B.s;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int j = blockIdx.x * kBlock + threadIdx.x;
    double phi = 0.0, nv[3] = {0.0, 0.0, 0.0}, Hs[6], gf[3] = {0.0, 0.0, 0.0};
    int i = -1;
    bool act = false;
    if (j < tp.nc) {
        i = tp.cnodes[j];
        double x[3];
#pragma unroll
        for (int d = 0; d < 3; d++) x[d] = tp.X[3 * i + d] + (double)B.u[3 * i + d];
        sdf_eval(s->ind, s->ind.c, x, false, phi, nv, Hs);
        act = phi < 0.0;
        if (s->mu_f > 0.0) {
            double fl[8], Hf[6], dd[3];
            const double zero[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int c = 0; c < 8; c++) fl[c] = B.fr[8 * j + c];
            if (fl[0] > 0.0) {
                friction_rel(fl, zero, dd);
                friction_eval(fl, dd, s->eps_f, gf, Hf);
                act = true;
            }
        }
    }
    double fv[3];
#pragma unroll
    for (int d = 0; d < 3; d++) fv[d] = act ? (phi < 0.0 ? -s->ind.k * phi * nv[d] : 0.0) - gf[d] : 0.0;
    const unsigned long long mask = __ballot(act);
    double sf[3];
#pragma unroll
    for (int d = 0; d < 3; d++) sf[d] = wave_sum(fv[d]);
    if (lane == 0) {
        wave_cnt[w] = __popcll(mask);
#pragma unroll
        for (int d = 0; d < 3; d++) wave_f[w][d] = sf[d];
    }
    __syncthreads();
    if (lists && act) {
        size_t slot = (size_t)blockIdx.x * kBlock + __popcll(mask & ((1ull << lane) - 1ull));
        for (int k = 0; k < w; k++) slot += wave_cnt[k];
        ids[slot] = i;
        phi_out[slot] = phi;
#pragma unroll
        for (int d = 0; d < 3; d++) f[3 * slot + d] = fv[d];
    }
    if (threadIdx.x == 0) {
        PatchHead h{};
        for (int k = 0; k < kWaves; k++) {
            h.count += wave_cnt[k];
#pragma unroll
            for (int d = 0; d < 3; d++) h.F[d] += wave_f[k][d];
        }
        heads[blockIdx.x] = h;
    }
}

// ---------------------------------------------------------------------------
// Node vectors between the device's numbering and the caller's, with pinned
// host memory in the path precision on the caller's side: consecutive threads
// touch consecutive host addresses, and device[c] is the device id of the
// caller's node c.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlock) void k_export_nodes(const int *device, const T *src, T *host, int n) {
    const int q = blockIdx.x * kBlock + threadIdx.x;
    if (q >= 3 * n) return;
    const int c = q / 3;
    host[q] = src[3 * device[c] + (q - 3 * c)];
}

// also: a second vector that takes the same values (also_zero: zeros), or null.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_import_nodes(const int *device, const T *host, T *dst, T *also,
                                                         bool also_zero, int n) {
    const int q = blockIdx.x * kBlock + threadIdx.x;
    if (q >= 3 * n) return;
    const int c = q / 3, to = 3 * device[c] + (q - 3 * c);
    const T v = host[q];
    dst[to] = v;
    if (also) also[to] = also_zero ? (T)0 : v;
}

// A job's state from pinned host memory.
__global__ void k_put_state(InstState *s, const InstState *from) {
    constexpr int kWords = sizeof(InstState) / 8;
    for (int q = threadIdx.x; q < kWords; q += blockDim.x)
        ((unsigned long long *)s)[q] = ((const unsigned long long *)from)[q];
}

// A job back at rest: zero displacement, velocity and predictor, and its new
// state from pinned host memory (one launch for three fills and a copy).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_restart(T *u, T *v, T *ut, int n3, InstState *s, const InstState *from) {
    const int q = blockIdx.x * kBlock + threadIdx.x;
    if (q < n3) u[q] = v[q] = ut[q] = (T)0;
    constexpr int kWords = sizeof(InstState) / 8;
    if (q < kWords) ((unsigned long long *)s)[q] = ((const unsigned long long *)from)[q];
}

// ---------------------------------------------------------------------------
// Outputs for data generation (one instance at its current state).
// k_tet_stress: one block per tile stages the tile's displacements in LDS;
// per tet F = I + G, the first Piola-Kirchhoff stress as in the element
// pass, the Cauchy stress sigma = P F^T / J (symmetrised; xx yy zz xy xz yz)
// and its von Mises value, written in FP64 at the tet's input index.
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(kBlock) void k_tet_stress(const Topo<T> *topos, const InstBufs<T> *bufs, int inst,
                                                       double *sigma, double *vm) {
    __shared__ __attribute__((aligned(32))) T su[kSw * kTileNodes];
    const BufsD<T> B = dev_view(bufs[inst]);
    const TopoD<T> tp = dev_view(topos[B.topo]);
    const int t = blockIdx.x;
    if (t >= tp.ntile) return;
    const T mu = (T)B.s->mu, lam = (T)B.s->lam;
    const int model = B.s->model;
    const int e0 = tp.tile_ent[t], ne = tp.tile_ent[t + 1] - e0;
    const int k0 = tp.tile_tet[t], nk = tp.tile_tet[t + 1] - k0;
    for (int l = threadIdx.x; l < ne; l += kBlock) {
        const int gid = tp.ent_node[e0 + l], sl = tp.ent_slot[e0 + l];
#pragma unroll
        for (int d = 0; d < 3; d++) su[kSw * sl + d] = B.u[3 * gid + d];
        su[kSw * sl + 3] = (T)0;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nk; k += kBlock) {
        int l[4];
        TetWords<T> tw;
        fetch_tet(tp, k0 + k, tw);
        const ElemGeo<T> geo = unpack_tet(tw, l);
        T wu[4][3];
        load_nodes(su, l, wu);
        T G[9];
        edge_gradient(wu, geo.Bm, G);
        const T Jm1 = det_minus_one(G);
        const T J = (T)1 + Jm1;
        const int id = tp.tet_id[k0 + k];
        double out[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
        double v = 0.0;
        if (J > (T)0) {
            T psi, mag, Pk[9], Mb[9], ka, kb, F[9];
            if (model == LAW_CR)
                Law<T, LAW_CR>::element(G, Jm1, J, mu, lam, psi, mag, Pk, Mb, ka, kb);
            else
                Law<T, LAW_NH>::element(G, Jm1, J, mu, lam, psi, mag, Pk, Mb, ka, kb);
#pragma unroll
            for (int c = 0; c < 9; c++) F[c] = G[c] + (c % 4 == 0 ? (T)1 : (T)0);
            double S[9];
#pragma unroll
            for (int i = 0; i < 3; i++)
#pragma unroll
                for (int j = 0; j < 3; j++)
                    S[3 * i + j] = ((double)Pk[3 * i] * F[3 * j] + (double)Pk[3 * i + 1] * F[3 * j + 1] +
                                    (double)Pk[3 * i + 2] * F[3 * j + 2]) / (double)J;
            out[0] = S[0];
            out[1] = S[4];
            out[2] = S[8];
            out[3] = 0.5 * (S[1] + S[3]);
            out[4] = 0.5 * (S[2] + S[6]);
            out[5] = 0.5 * (S[5] + S[7]);
            const double a = out[0] - out[1], b = out[1] - out[2], c = out[2] - out[0];
            v = sqrt(0.5 * (a * a + b * b + c * c) + 3.0 * (out[3] * out[3] + out[4] * out[4] + out[5] * out[5]));
        } else {
            v = NAN;
#pragma unroll
            for (int c = 0; c < 6; c++) out[c] = NAN;
        }
        if (sigma)
#pragma unroll
            for (int c = 0; c < 6; c++) sigma[6 * (size_t)id + c] = out[c];
        if (vm) vm[id] = v;
    }
}

// max_i |u_i| and mean_i |u_i| of one instance (one block, FP64 sums; out in
// pinned host memory).
template <typename T>
__global__ __launch_bounds__(1024) void k_disp_stats(const Topo<T> *topos, const InstBufs<T> *bufs, int inst,
                                                     double *out) {
    __shared__ double smax[16], ssum[16];
    const BufsD<T> B = dev_view(bufs[inst]);
    const int n = topos[B.topo].n;
    double mx = 0.0, sum = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        const double x = B.u[3 * i], y = B.u[3 * i + 1], z = B.u[3 * i + 2];
        const double a = sqrt(x * x + y * y + z * z);
        mx = fmax(mx, a);
        sum += a;
    }
    sum = wave_sum(sum);
    mx = -wave_min(-mx);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    if (lane == 0) {
        smax[wv] = mx;
        ssum[wv] = sum;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double m2 = 0.0, s2 = 0.0;
        for (int k = 0; k < (int)(blockDim.x >> 6); k++) {
            m2 = fmax(m2, smax[k]);
            s2 += ssum[k];
        }
        out[0] = m2;
        out[1] = n > 0 ? s2 / n : 0.0;
    }
}

// ---------------------------------------------------------------------------
// Mesh set-up kernels.
// ---------------------------------------------------------------------------
// Rest volume check (FP64): records the first tet with det D_m <= 0.
__global__ __launch_bounds__(kBlock) void k_check_volumes(const double *X, const int *tet, int m, int *bad) {
    const int e = blockIdx.x * kBlock + threadIdx.x;
    if (e >= m) return;
    const int v0 = tet[4 * e];
    double D[9];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const int va = tet[4 * e + a + 1];
#pragma unroll
        for (int i = 0; i < 3; i++) D[3 * i + a] = X[3 * va + i] - X[3 * v0 + i];
    }
    const double det = D[0] * (D[4] * D[8] - D[5] * D[7]) - D[1] * (D[3] * D[8] - D[5] * D[6]) +
                       D[2] * (D[3] * D[7] - D[4] * D[6]);
    if (!(det > 0.0)) atomicMin(bad, e);
}

// Rest constants per tet in tile order (FP64, stored in the path precision):
// D_m = [X1-X0, X2-X0, X3-X0], D_m^-1 by cofactors, V = |det D_m| / 6, from
// the tet's nodes in device vertex order (tnodes, 4 per tet in tile order;
// any reordering of the input's vertices: F = D_s D_m^-1 does not depend on
// it, and the input orientation is checked by k_check_volumes); with the
// tet's packed local node slots.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_rest_constants(const double *X, const int *tnodes, const uint32_t *loc,
                                                           int m, TetRec<T> *rec) {
    const int k = blockIdx.x * kBlock + threadIdx.x;
    if (k >= m) return;
    const int *tet = tnodes + 4 * (size_t)k;
    const int v0 = tet[0];
    double D[9];
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const int va = tet[a + 1];
#pragma unroll
        for (int i = 0; i < 3; i++) D[3 * i + a] = X[3 * va + i] - X[3 * v0 + i];
    }
    const double c00 = D[4] * D[8] - D[5] * D[7], c01 = D[5] * D[6] - D[3] * D[8], c02 = D[3] * D[7] - D[4] * D[6];
    const double det = D[0] * c00 + D[1] * c01 + D[2] * c02;
    const double id = 1.0 / det;
    const double inv[9] = {c00 * id, (D[2] * D[7] - D[1] * D[8]) * id, (D[1] * D[5] - D[2] * D[4]) * id,
                           c01 * id, (D[0] * D[8] - D[2] * D[6]) * id, (D[2] * D[3] - D[0] * D[5]) * id,
                           c02 * id, (D[1] * D[6] - D[0] * D[7]) * id, (D[0] * D[4] - D[1] * D[3]) * id};
    TetRec<T> r{};
#pragma unroll
    for (int c = 0; c < 9; c++) r.Bm[c] = (T)inv[c];
    r.V = (T)(fabs(det) / 6.0);
    r.loc = loc[k];
    rec[k] = r;
}

// Boundary faces by hashing the sorted node triple (21 bits per id) of each
// of the 4m faces into an open-addressing table; faces seen once are on the
// boundary.
__device__ __forceinline__ unsigned long long face_key(const int *tet, int e, int f) {
    int a = tet[4 * e + ((f + 1) & 3)], b = tet[4 * e + ((f + 2) & 3)], c = tet[4 * e + ((f + 3) & 3)];
    int t;
    if (a > b) { t = a; a = b; b = t; }
    if (b > c) { t = b; b = c; c = t; }
    if (a > b) { t = a; a = b; b = t; }
    return ((unsigned long long)a << 42) | ((unsigned long long)b << 21) | (unsigned long long)c;
}

// Slot hash of a face key: the 64-bit finaliser (fmix64) of Austin Appleby's
// public-domain MurmurHash3, with its published shift and multiplier constants.
__device__ __forceinline__ unsigned face_hash(unsigned long long k) {
    k ^= k >> 33;
    k *= 0xff51afd7ed558ccdull;
    k ^= k >> 33;
    k *= 0xc4ceb9fe1a85ec53ull;
    k ^= k >> 33;
    return (unsigned)k;
}

__global__ __launch_bounds__(kBlock) void k_faces_insert(const int *tet, int m, unsigned long long *keys,
                                                         unsigned *cnt, unsigned mask) {
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= 4 * m) return;
    const unsigned long long k = face_key(tet, t >> 2, t & 3);
    unsigned h = face_hash(k) & mask;
    for (;;) {   // load factor <= 1/2: a free or matching slot is always found
        const unsigned long long prev = atomicCAS(keys + h, ~0ull, k);
        if (prev == ~0ull || prev == k) {
            atomicAdd(cnt + h, 1u);
            return;
        }
        h = (h + 1) & mask;
    }
}

__global__ __launch_bounds__(kBlock) void k_faces_mark(const int *tet, int m, const unsigned long long *keys,
                                                       const unsigned *cnt, unsigned mask, uint8_t *surf) {
    const int t = blockIdx.x * kBlock + threadIdx.x;
    if (t >= 4 * m) return;
    const int e = t >> 2, f = t & 3;
    const unsigned long long k = face_key(tet, e, f);
    unsigned h = face_hash(k) & mask;
    while (keys[h] != k) h = (h + 1) & mask;   // the key was inserted
    if (cnt[h] == 1u) {
        surf[tet[4 * e + ((f + 1) & 3)]] = 1;
        surf[tet[4 * e + ((f + 2) & 3)]] = 1;
        surf[tet[4 * e + ((f + 3) & 3)]] = 1;
    }
}

// One block: eligible = surface and not fixed; ascending compaction and the
// node -> contact slot map.
__global__ __launch_bounds__(1024) void k_compact_eligible(const uint8_t *surf, const uint8_t *fixed, int n,
                                                           uint8_t *elig, int *list, int *cidx, int *count) {
    __shared__ int wave_cnt[16];
    __shared__ int base_s;
    if (threadIdx.x == 0) base_s = 0;
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int start = 0; start < n; start += 1024) {
        const int i = start + threadIdx.x;
        const bool act = i < n && surf[i] && !fixed[i];
        const unsigned long long mask = __ballot(act);
        if (lane == 0) wave_cnt[w] = __popcll(mask);
        __syncthreads();
        int off = base_s;
        for (int k = 0; k < w; k++) off += wave_cnt[k];
        if (i < n) {
            elig[i] = act ? 1 : 0;
            const int slot = off + __popcll(mask & ((1ull << lane) - 1ull));
            cidx[i] = act ? slot : -1;
            if (act) list[slot] = i;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int tot = 0;
            for (int k = 0; k < 16; k++) tot += wave_cnt[k];
            base_s += tot;
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) *count = base_s;
}

}  // namespace fem

// kcm_kernels.hip -- gfx950 kernels of one KCM iteration.
//
//   k_tau       one thread per joint: joint torques of the pending forces,
//               tau_k = u_k . (T_k - p_k x F_k) (eqs KCM_01-KCM_06), with the
//               wrench of later atom workgroups from a suffix (row) scan
//               (eq 04_9).
//   k_stepfk    one thread per joint: the compliance step (eq KCM_07), then
//               forward kinematics of the new angles as an ordered prefix
//               scan of rigid transforms inside each joint block (eqs
//               kin_02-kin_04, r1; prefix computation item 1 of Sec. 3.5).
//   k_place     one thread per atom: link transforms (products of the
//               earlier joint blocks composed in front of the block-local
//               ones), r_a = G_link(a) r0_a, per-workgroup bounding box of
//               the new positions.
//   k_cellkey   one thread per atom: the cell grid of Sec. 3.2 sized from
//               that bounding box (in every workgroup of a small chain, in
//               k_grid before it for a large one), cell key, count and the
//               atom's place among its cell's arrivals.
//   k_cellscan  one workgroup per 4096 cells: exclusive scan of the counts
//               inside the chunk, and its total.
//   (k_scatter and k_rank add the chunk offsets; k_rank writes the starts.)
//   k_scatter   one thread per atom: counting-sort scatter by cell key.
//   k_rank      one thread per atom: stable slot inside the cell, gather.
//   k_force     one wave per atom, atoms in cell order: stencil candidates
//               in FP64, Coulomb + LJ (eqs 02-03_9), solvation neighbours in
//               LDS, and the SASA enumeration of Algorithm 1 with the C-state
//               rules (Sec. 3.4): coverage counts with four samples per lane,
//               the displaced tests of critical samples and of exposed ones
//               from a queue of (sample, neighbour) pairs.  Solvation events
//               are scattered as fixed-point integers.
//   k_wrench    one thread per atom: wrench (F, r x F), the suffix sum inside
//               the workgroup and the workgroup-local part of each torque.
//   k_chain     one workgroup per chain: all of these but k_force, for calls of
//               short or many chains, whose iterations are then two launches.
#include "kcm_internal.h"

#include <float.h>
#include <math.h>

#include <algorithm>

namespace kcm {

constexpr int WAVE = 64;
constexpr double PI_D = 3.14159265358979323846;
// Half width of the FP32 decision band of the mixed form: a sample test whose
// FP32 value lies this close to its threshold is decided again in FP64.  The
// FP32 error of the tested quantity stays below ~5e-6 A for offsets < 16 A.
constexpr float MIXED_BAND = 4.0e-5f;

// Loads, stores and atomics through a pointer of unknown address space are
// flat instructions, which count against the LDS counter as well as the
// vector-memory one: every LDS wait then also waits for them.  The device
// arrays of the force kernel are all in global memory, and it reaches them
// through these global-address-space views (plain pointers in the host
// pass, which only checks the device code).
#if defined(__HIP_DEVICE_COMPILE__)
template <typename T> using gptr = __attribute__((address_space(1))) T *;
#else
template <typename T> using gptr = T *;
#endif
template <typename T> __device__ __forceinline__ gptr<T> glob(T *p) { return (gptr<T>)p; }

// ---------------------------------------------------------------------------
// moves between the lanes of a wave
// ---------------------------------------------------------------------------
// A shuffle is two LDS permutes per double, and one CU's LDS takes about ten
// cycles for each: the scans and reductions of the chain kernels were bound by
// them.  The moves below stay in the vector unit where the
// pattern allows it: shifts by one lane and rotations inside a row of 16 are
// data-parallel modifiers, swaps of half waves and of rows are single
// instructions.  They carry the same values to the same lanes.
template <int CTRL> __device__ __forceinline__ int dpp(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true); }
template <int CTRL> __device__ __forceinline__ double dpp(double x)
{
    return __hiloint2double(dpp<CTRL>(__double2hiint(x)), dpp<CTRL>(__double2loint(x)));
}
constexpr int DPP_WAVE_SHL1 = 0x130, DPP_WAVE_SHR1 = 0x138, DPP_ROW_ROR = 0x120, DPP_ROW_SHL = 0x100, DPP_ROW_SHR = 0x110;
constexpr int DPP_QUAD_XOR1 = 0xb1, DPP_QUAD_XOR2 = 0x4e;
// the lower half of the wave in both halves (UPPER: the upper one), and the
// even rows of 16 in both rows of each half (UPPER: the odd ones)
template <bool UPPER> __device__ __forceinline__ int both_halves(int x)
{
    return (int)__builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false)[UPPER];
}
template <bool UPPER> __device__ __forceinline__ int both_rows(int x)
{
    return (int)__builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false)[UPPER];
}
template <bool UPPER> __device__ __forceinline__ double both_halves(double x)
{
    return __hiloint2double(both_halves<UPPER>(__double2hiint(x)), both_halves<UPPER>(__double2loint(x)));
}
template <bool UPPER> __device__ __forceinline__ double both_rows(double x)
{
    return __hiloint2double(both_rows<UPPER>(__double2hiint(x)), both_rows<UPPER>(__double2loint(x)));
}
// lane l takes the value of lane l - d (lanes below d: anything); d a power of two, known when compiled
__device__ __forceinline__ double from_below(double x, int d)
{
    if (d == 1) return dpp<DPP_WAVE_SHR1>(x);
    if (d == 2) return dpp<DPP_WAVE_SHR1>(dpp<DPP_WAVE_SHR1>(x));
    if (d == 32) return both_halves<false>(x);
    return __shfl_up(x, d, WAVE);
}
// lane l takes the value of lane l + d (the last d lanes: anything)
__device__ __forceinline__ double from_above(double x, int d)
{
    if (d == 1) return dpp<DPP_WAVE_SHL1>(x);
    if (d == 2) return dpp<DPP_WAVE_SHL1>(dpp<DPP_WAVE_SHL1>(x));
    if (d == 32) return both_halves<true>(x);
    return __shfl_down(x, d, WAVE);
}
// the lanes where p holds (from the compare's own mask, where the library's
// ballot goes through a 0/1 register and a second compare)
__device__ __forceinline__ unsigned long long ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }
// set bits of m in the lanes below this one (the hardware's masked bit count)
__device__ __forceinline__ int count_below(unsigned long long m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}
// op over the wave in every lane, as the butterfly over lane distances 32, 16,
// ..., 1 takes it: below 16 the values repeat with the last distance inside a
// row, so a rotation by half of it brings the partner's
template <typename T, typename Op> __device__ __forceinline__ T wave_all(T v, Op op)
{
    v = op(both_halves<false>(v), both_halves<true>(v));
    v = op(both_rows<false>(v), both_rows<true>(v));
    v = op(v, dpp<DPP_ROW_ROR + 8>(v));
    v = op(v, dpp<DPP_ROW_ROR + 4>(v));
    v = op(v, dpp<DPP_ROW_ROR + 2>(v));
    return op(v, dpp<DPP_ROW_ROR + 1>(v));
}

// inclusive prefix sum over the wave: inside rows of 16, then the last lane of
// each row into the next, then of the lower half into the upper
__device__ __forceinline__ int wave_scan_i(int x)
{
    x += dpp<DPP_ROW_SHR + 1>(x);
    x += dpp<DPP_ROW_SHR + 2>(x);
    x += dpp<DPP_ROW_SHR + 4>(x);
    x += dpp<DPP_ROW_SHR + 8>(x);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);
    return x;
}

// Several sums at once: where a butterfly adds the two halves of one value in
// all lanes, the halves of two values are exchanged first and one add serves
// both.  Each value's sum is the one wave_all gives, in the lanes named.
__device__ __forceinline__ void swap_halves(int &a, int &b)
{
    const auto r = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
    a = (int)r[0];
    b = (int)r[1];
}
__device__ __forceinline__ void swap_rows(int &a, int &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap((unsigned)a, (unsigned)b, false, false);
    a = (int)r[0];
    b = (int)r[1];
}
__device__ __forceinline__ double sum_halves(double a, double b)
{
    int ah = __double2hiint(a), al = __double2loint(a), bh = __double2hiint(b), bl = __double2loint(b);
    swap_halves(ah, bh);
    swap_halves(al, bl);
    return __hiloint2double(ah, al) + __hiloint2double(bh, bl);
}
__device__ __forceinline__ double sum_rows(double a, double b)
{
    int ah = __double2hiint(a), al = __double2loint(a), bh = __double2hiint(b), bl = __double2loint(b);
    swap_rows(ah, bh);
    swap_rows(al, bl);
    return __hiloint2double(ah, al) + __hiloint2double(bh, bl);
}
__device__ __forceinline__ int from_xor4(int x)
{
    const int t = __builtin_amdgcn_update_dpp(0, x, DPP_ROW_SHL + 4, 0xf, 0x5, false);
    return __builtin_amdgcn_update_dpp(t, x, DPP_ROW_SHR + 4, 0xf, 0xa, false);
}
// a in lane 0, b in lane 32, c in lane 16, d in lane 48, e in lane 8: 37
// instructions in place of 120 for five sums in all lanes
__device__ __forceinline__ double wave_sum5(double a, double b, double c, double d, double e)
{
    const double p = sum_rows(sum_halves(a, b), sum_halves(c, d));
    double v = both_halves<false>(e) + both_halves<true>(e);
    v = both_rows<false>(v) + both_rows<true>(v);
    const bool up = threadIdx.x & 8;
    double z = (up ? v : p) + dpp<DPP_ROW_ROR + 8>(up ? p : v);
    z += __hiloint2double(from_xor4(__double2hiint(z)), from_xor4(__double2loint(z)));
    z += dpp<DPP_QUAD_XOR2>(z);
    return z + dpp<DPP_QUAD_XOR1>(z);
}
// a in lane 0, b in lane 32, c in lane 16, d in lane 48
__device__ __forceinline__ int wave_sum4_i(int a, int b, int c, int d)
{
    swap_halves(a, b);
    swap_halves(c, d);
    int p = a + b, q = c + d;
    swap_rows(p, q);
    p += q;
    p += dpp<DPP_ROW_ROR + 8>(p);
    p += dpp<DPP_ROW_ROR + 4>(p);
    p += dpp<DPP_ROW_ROR + 2>(p);
    return p + dpp<DPP_ROW_ROR + 1>(p);
}

// The smaller and the larger of two numbers.  The library's calls first quiet
// signalling NaNs, one more instruction per argument that went between lanes.
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ double min_num(double a, double b)
{
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ double max_num(double a, double b)
{
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
#else
__device__ double min_num(double a, double b);
__device__ double max_num(double a, double b);
#endif
__device__ __forceinline__ double lane_value(double x, int l)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
}
// The box [lo, hi] over the wave, the same in every lane: minima of the six
// numbers lo and -hi, reduced together as in wave_sum5 (60 instructions in
// place of 280 for six butterflies).
__device__ __forceinline__ void wave_box(double (&lo)[3], double (&hi)[3])
{
    auto halves = [](double a, double b) {
        int ah = __double2hiint(a), al = __double2loint(a), bh = __double2hiint(b), bl = __double2loint(b);
        swap_halves(ah, bh);
        swap_halves(al, bl);
        return min_num(__hiloint2double(ah, al), __hiloint2double(bh, bl));
    };
    auto rows = [](double a, double b) {
        int ah = __double2hiint(a), al = __double2loint(a), bh = __double2hiint(b), bl = __double2loint(b);
        swap_rows(ah, bh);
        swap_rows(al, bl);
        return min_num(__hiloint2double(ah, al), __hiloint2double(bh, bl));
    };
    const double p = rows(halves(lo[0], lo[1]), halves(lo[2], -hi[0]));
    double v = halves(-hi[1], -hi[2]);
    v = min_num(both_rows<false>(v), both_rows<true>(v));
    const bool up = threadIdx.x & 8;
    double z = min_num(up ? v : p, dpp<DPP_ROW_ROR + 8>(up ? p : v));
    z = min_num(z, __hiloint2double(from_xor4(__double2hiint(z)), from_xor4(__double2loint(z))));
    z = min_num(z, dpp<DPP_QUAD_XOR2>(z));
    z = min_num(z, dpp<DPP_QUAD_XOR1>(z));
    lo[0] = lane_value(z, 0);
    lo[1] = lane_value(z, 32);
    lo[2] = lane_value(z, 16);
    hi[0] = -lane_value(z, 48);
    hi[1] = -lane_value(z, 8);
    hi[2] = -lane_value(z, 40);
}

// Inside a condition on the lane: the compiler then runs the branch under the
// execution mask, where it would compute for all lanes and select each word of
// each result (two instructions per double).
__device__ __forceinline__ void masked_branch() { asm volatile(""); }

// A barrier for what the workgroup shares in LDS.  __syncthreads() also waits
// for every load and store under way to global memory, a thousand cycles where
// a store has just gone out.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ---------------------------------------------------------------------------
// rigid transforms (rotation R row-major, translation t): x -> R x + t
// ---------------------------------------------------------------------------
struct Xf {
    double r[9];
    double t[3];
};

__device__ __forceinline__ Xf xf_identity()
{
    Xf x;
#pragma unroll
    for (int k = 0; k < 9; ++k) x.r[k] = (k % 4 == 0) ? 1.0 : 0.0;
    x.t[0] = x.t[1] = x.t[2] = 0.0;
    return x;
}

// (A o B)(x) = A(B(x))
__device__ __forceinline__ Xf xf_mul(const Xf &A, const Xf &B)
{
    Xf C;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
#pragma unroll
        for (int j = 0; j < 3; ++j)
            C.r[3 * i + j] = A.r[3 * i] * B.r[j] + A.r[3 * i + 1] * B.r[3 + j] + A.r[3 * i + 2] * B.r[6 + j];
        C.t[i] = A.r[3 * i] * B.t[0] + A.r[3 * i + 1] * B.t[1] + A.r[3 * i + 2] * B.t[2] + A.t[i];
    }
    return C;
}

__device__ __forceinline__ Xf xf_from_below(const Xf &x, int d)
{
    Xf y;
#pragma unroll
    for (int k = 0; k < 9; ++k) y.r[k] = from_below(x.r[k], d);
#pragma unroll
    for (int k = 0; k < 3; ++k) y.t[k] = from_below(x.t[k], d);
    return y;
}

template <typename P> __device__ __forceinline__ void xf_store(P p, const Xf &x)
{
#pragma unroll
    for (int k = 0; k < 9; ++k) p[k] = x.r[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) p[9 + k] = x.t[k];
}

template <typename P> __device__ __forceinline__ Xf xf_load(P p)
{
    Xf x;
#pragma unroll
    for (int k = 0; k < 9; ++k) x.r[k] = p[k];
#pragma unroll
    for (int k = 0; k < 3; ++k) x.t[k] = p[9 + k];
    return x;
}

__device__ __forceinline__ int link_of_atom(int a)
{
    const int res = a / APR, slot = a - res * APR;
    return 2 * res + (slot < 2 ? 0 : (slot < 8 ? 1 : 2));
}

// ---------------------------------------------------------------------------
// block-wide helpers (blockDim.x a multiple of 64, at most 1024)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v)
{
    return wave_all(v, [](double a, double b) { return a + b; });
}
__device__ __forceinline__ double wave_max(double v)
{
    return wave_all(v, [](double a, double b) { return max_num(a, b); });
}
__device__ __forceinline__ int wave_sum_i(int v)
{
    return wave_all(v, [](int a, int b) { return a + b; });
}

// Sum of K doubles over the block; the result is returned to every thread.
// Fixed reduction order, so it is deterministic.  scratch: [16][K].
template <int K>
__device__ void block_sum(double (&v)[K], double *scratch)
{
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = wave_sum(v[k]);
    lds_barrier();
    if (lane == 0)
        for (int k = 0; k < K; ++k) scratch[w * K + k] = v[k];
    lds_barrier();
#pragma unroll
    for (int k = 0; k < K; ++k) {
        double s = 0.0;
        for (int i = 0; i < nw; ++i) s += scratch[i * K + k];
        v[k] = s;
    }
    lds_barrier();
}

// The largest v over the block and whether any thread has bad set, in every
// thread.  scratch, s_bad: one entry per wave, not in use.
__device__ __forceinline__ double block_max_any(double v, bool &bad, double *scratch, int *s_bad)
{
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
    v = wave_max(v);
    bad = __any(bad);
    if (lane == 0) {
        scratch[w] = v;
        s_bad[w] = bad;
    }
    lds_barrier();
    for (int i = 0; i < nw; ++i) {
        v = fmax(v, scratch[i]);
        bad = bad || s_bad[i];
    }
    return v;
}

// Exclusive prefix sum of one int per thread over the block; *total gets the sum.
__device__ int block_excl_scan(int v, int *scratch, int *total)
{
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE, nw = blockDim.x / WAVE;
    const int x = wave_scan_i(v);
    lds_barrier();
    if (lane == WAVE - 1) scratch[w] = x;
    lds_barrier();
    int base = 0, tot = 0;
    for (int i = 0; i < nw; ++i) {
        if (i < w) base += scratch[i];
        tot += scratch[i];
    }
    lds_barrier();
    *total = tot;
    return base + x - v;
}


__device__ __forceinline__ int find_block_owner(const int32_t *off, int n, int b)
{
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (off[mid] <= b) lo = mid; else hi = mid;
    }
    return lo;
}

// The chain of workgroup b, by the map of the launch's workgroups to chains (or
// a search where there is none), and its first workgroup.
struct Owner {
    ChainDev *cd;
    int chain, first;
};
__device__ __forceinline__ Owner owner_of(const Batch &bt, const int32_t *map, const int32_t *off, int b)
{
    if (bt.n_chains == 1) return {bt.only, 0, 0};
    const int c = map ? map[b] : find_block_owner(off, bt.n_chains, b);
    return {bt.table[c], c, off[c]};
}
// A chain's flags and grid lie at fixed places behind its descriptor: their
// loads need not wait for its pointers.
__device__ __forceinline__ ChainStats *stats_of(const ChainDev *cd)
{
    return reinterpret_cast<ChainStats *>(reinterpret_cast<char *>(const_cast<ChainDev *>(cd)) + STATS_OFFSET);
}
__device__ __forceinline__ Grid *grid_of(const ChainDev *cd)
{
    return reinterpret_cast<Grid *>(reinterpret_cast<char *>(const_cast<ChainDev *>(cd)) + GRID_OFFSET);
}

// The kernels after the step run a chain iff the step kept it running and its
// grid for this iteration could be sized.
__device__ __forceinline__ bool running(const ChainStats *st) { return (st->run != 0) & (st->grid_bad == 0); }

__device__ __forceinline__ int cell_of(const Grid &g, const double4 &r)
{
    int cx = (int)floor((r.x - g.origin[0]) * g.inv_cell);
    int cy = (int)floor((r.y - g.origin[1]) * g.inv_cell);
    int cz = (int)floor((r.z - g.origin[2]) * g.inv_cell);
    cx = min(max(cx, 0), g.dims[0] - 1);
    cy = min(max(cy, 0), g.dims[1] - 1);
    cz = min(max(cz, 0), g.dims[2] - 1);
    return (cz * g.dims[1] + cy) * g.dims[0] + cx;
}

constexpr double GRID_MARGIN = 2.0;  // A added around the bounding box of the placed atoms
constexpr int LINKS_PER_BLOCK = 56;  // links touched by ATOM_BLOCK consecutive atoms (at most 53)

// First atom moved by joint j: the first atom of link j+1 (C-alpha for phi,
// C for psi).
__device__ __forceinline__ int first_atom_of_joint(int j) { return APR * (j >> 1) + ((j & 1) ? 8 : 2); }
__device__ __forceinline__ int first_atom_of_link(int l) { return l == 0 ? 0 : first_atom_of_joint(l - 1); }

__device__ __forceinline__ Xf xf_shfl_idx(const Xf &x, int src)
{
    Xf y;
#pragma unroll
    for (int k = 0; k < 9; ++k) y.r[k] = __shfl(x.r[k], src, WAVE);
#pragma unroll
    for (int k = 0; k < 3; ++k) y.t[k] = __shfl(x.t[k], src, WAVE);
    return y;
}

// The current axis (u_j, p_j) of joint j from the transform G of link j + 1.
template <typename P>
__device__ __forceinline__ void fk_emit(const Xf &G, int j, const double4 &u0, const double4 &p0, P jcur)
{
    // the fused steps written out: every kernel that calls this rounds alike
    auto row = [&](int k, const double4 &v) {
        return fma(G.r[k + 2], v.z, fma(G.r[k], v.x, G.r[k + 1] * v.y));
    };
    double4 u, p;
    u.x = row(0, u0);
    u.y = row(3, u0);
    u.z = row(6, u0);
    u.w = 0.0;
    p.x = row(0, p0) + G.t[0];
    p.y = row(3, p0) + G.t[1];
    p.z = row(6, p0) + G.t[2];
    p.w = 0.0;
    jcur[2 * j] = u;
    jcur[2 * j + 1] = p;
}

// Rodrigues rotation about unit u by angle (th - pi) and the translation that
// keeps the axis point p fixed.
__device__ __forceinline__ Xf joint_xf_of(const double4 &u, const double4 &p, double th)
{
    double s, c;
    sincos(th - PI_D, &s, &c);
    const double k = 1.0 - c;
    Xf x;
    x.r[0] = c + u.x * u.x * k;       x.r[1] = u.x * u.y * k - u.z * s; x.r[2] = u.x * u.z * k + u.y * s;
    x.r[3] = u.y * u.x * k + u.z * s; x.r[4] = c + u.y * u.y * k;       x.r[5] = u.y * u.z * k - u.x * s;
    x.r[6] = u.z * u.x * k - u.y * s; x.r[7] = u.z * u.y * k + u.x * s; x.r[8] = c + u.z * u.z * k;
#pragma unroll
    for (int i = 0; i < 3; ++i) x.t[i] = ((&p.x)[i]) - (x.r[3 * i] * p.x + x.r[3 * i + 1] * p.y + x.r[3 * i + 2] * p.z);
    return x;
}

// A chain's descriptor as the chain kernels use it, read once at their start
// while nothing is stored yet: into scalar registers, where a later look would
// be a vector load (the stores might change the descriptor, for all the
// compiler knows) with a few hundred cycles of latency each.
struct ChainView {
    int n_atoms, n_joints, n_chi, n_bb_blocks, cap_cells, precision, step_rule;
    double cutoff, kappa, max_step, delta_r, cell_min, roff_max;
    gptr<double> theta, dtheta, tau, xform_loc, blk_xf, tmax_part, bbox_part, wrench_part;
    gptr<uint8_t> mask;
    gptr<double4> joint0, jcur, r0, r, aparam, s_r, s_p, f_pair, e_atom;
    gptr<int32_t> bad_part, cell_key, cell_count, cell_start, cell_local, scan_part, s_tmp, s_idx;
    gptr<long long> f_cav;
    __device__ __forceinline__ explicit ChainView(const ChainDev *d)
        : n_atoms(d->n_atoms), n_joints(d->n_joints), n_chi(d->n_chi), n_bb_blocks(d->n_bb_blocks),
          cap_cells(d->cap_cells), precision(d->precision), step_rule(d->step_rule), cutoff(d->cutoff),
          kappa(d->kappa), max_step(d->max_step), delta_r(d->delta_r), cell_min(d->cell_min), roff_max(d->roff_max),
          theta(glob(d->theta)), dtheta(glob(d->dtheta)), tau(glob(d->tau)), xform_loc(glob(d->xform_loc)),
          blk_xf(glob(d->blk_xf)), tmax_part(glob(d->tmax_part)), bbox_part(glob(d->bbox_part)),
          wrench_part(glob(d->wrench_part)), mask(glob(d->mask)), joint0(glob(d->joint0)), jcur(glob(d->jcur)),
          r0(glob(d->r0)), r(glob(d->r)), aparam(glob(d->aparam)), s_r(glob(d->s_r)), s_p(glob(d->s_p)),
          f_pair(glob(d->f_pair)), e_atom(glob(d->e_atom)), bad_part(glob(d->bad_part)), cell_key(glob(d->cell_key)),
          cell_count(glob(d->cell_count)), cell_start(glob(d->cell_start)), cell_local(glob(d->cell_local)),
          scan_part(glob(d->scan_part)), s_tmp(glob(d->s_tmp)), s_idx(glob(d->s_idx)), f_cav(glob(d->f_cav))
    {
    }
};
// Loads that are done where this stands: all those named go out together, ahead
// of the flags that say whether they are needed (they are of memory that is
// there either way), in place of one latency after the other.
// (The eight small kernels of an iteration, which are bound by such latencies:
// 43.4 us before, 38.8 us with these and LDS barriers, for 10,000 atoms.)
__device__ __forceinline__ void loaded_one(double v) { asm volatile("" : : "v"(v)); }
__device__ __forceinline__ void loaded_one(long long v) { asm volatile("" : : "v"(v)); }
__device__ __forceinline__ void loaded_one(int v) { asm volatile("" : : "v"(v)); }
__device__ __forceinline__ void loaded_one(const double4 &v) { asm volatile("" : : "v"(v.x), "v"(v.y), "v"(v.z)); }
template <typename... T> __device__ __forceinline__ void loaded(const T &...v) { (loaded_one(v), ...); }

// What a chain's grid is sized by.
struct GridRule {
    double reach_len, cell, inv_cell;  // interaction reach, first cell edge
    int cap_cells;
};
template <typename Chain>
__device__ __forceinline__ GridRule grid_rule(const Chain *cd)
{
    const double reach_len = fmax(cd->cutoff, 2.0 * cd->roff_max + cd->delta_r) + 1e-7;
    const double cell = fmax(cd->cell_min, reach_len / MAX_REACH);
    return {reach_len, cell, 1.0 / cell, cd->cap_cells};
}
// The grid of Sec. 3.2 for the bounding box [lo, hi] of the placed atoms, plus a
// margin, by a whole wave: lane k < 3 brings axis k's bounds, the others axis
// 2's, and all get the grid; ok stays true iff it could be sized within the
// capacity.  The cell edge starts at max(cell_min, reach / MAX_REACH) and grows
// until the grid fits the chain's cell capacity.
__device__ __forceinline__ Grid size_grid(const GridRule &rule, double lo, double hi, bool &ok)
{
    const double L = lo - GRID_MARGIN, H = hi + GRID_MARGIN, ext = H - L;
    ok = !__any(!(ok && isfinite(L) && isfinite(H) && H >= L && ext < 1e7));
    Grid g;
    g.reach_len = rule.reach_len;
    g.cell = rule.cell;
    g.inv_cell = rule.inv_cell;
    long long dims[3] = {1, 1, 1};
    for (int it = 0; ok && it < 200; ++it) {
        const long long d = (long long)floor(ext / g.cell) + 1;
        const int d_lo = (int)d, d_hi = (int)(d >> 32);
#pragma unroll
        for (int k = 0; k < 3; ++k)
            dims[k] = ((long long)__builtin_amdgcn_readlane(d_hi, k) << 32) | (unsigned)__builtin_amdgcn_readlane(d_lo, k);
        if (dims[0] * dims[1] * dims[2] <= rule.cap_cells) break;
        g.cell *= 1.2599210498948732;
        g.inv_cell = 1.0 / g.cell;
    }
    ok = ok && dims[0] * dims[1] * dims[2] <= rule.cap_cells;
#pragma unroll
    for (int k = 0; k < 3; ++k) { g.origin[k] = ok ? lane_value(L, k) : 0.0; g.dims[k] = ok ? (int)dims[k] : 1; }
    g.reach = max(1, (int)ceil(g.reach_len / g.cell - 1e-9));
    g.n_cells = ok ? (int)(dims[0] * dims[1] * dims[2]) : 1;
    g.pad = 0;
    return g;
}
// lane k < 3: v[k], the others: v[2]
__device__ __forceinline__ double axis_of_lane(const double (&v)[3])
{
    const int lane = threadIdx.x & (WAVE - 1);
    return lane == 0 ? v[0] : lane == 1 ? v[1] : v[2];
}

// The grid from the per-workgroup bounding boxes, block-wide (any block size);
// returns false (and a one-cell grid) when the box is not finite or cannot be
// covered.  s_red: [nw * 6].
__device__ bool grid_from_parts(const ChainDev *cd, Grid *out, double *s_red, int *s_ok)
{
    const int n = cd->n_atoms;
    const int nblk = (n + ATOM_BLOCK - 1) / ATOM_BLOCK;
    const int tid = threadIdx.x, nt = blockDim.x, lane = tid & (WAVE - 1), w = tid / WAVE, nw = nt / WAVE;
    double lo[3] = {DBL_MAX, DBL_MAX, DBL_MAX}, hi[3] = {-DBL_MAX, -DBL_MAX, -DBL_MAX};
    bool fin = true;
    for (int b = tid; b < nblk; b += nt)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double l = cd->bbox_part[6 * b + k], h = cd->bbox_part[6 * b + 3 + k];
            fin = fin && isfinite(l) && isfinite(h);
            lo[k] = fmin(lo[k], l);
            hi[k] = fmax(hi[k], h);
        }
    wave_box(lo, hi);
    const bool bad_w = __any(!fin);
    if (tid == 0) *s_ok = 1;
    __syncthreads();
    if (lane == 0) {
        for (int k = 0; k < 3; ++k) { s_red[w * 6 + k] = lo[k]; s_red[w * 6 + 3 + k] = hi[k]; }
        if (bad_w) *s_ok = 0;
    }
    __syncthreads();
    if (w == 0) {
        // wave 0 reduces the wave partials, lane i holding wave i's
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            lo[k] = lane < nw ? s_red[lane * 6 + k] : DBL_MAX;
            hi[k] = lane < nw ? s_red[lane * 6 + 3 + k] : -DBL_MAX;
        }
        wave_box(lo, hi);
        bool ok = *s_ok != 0;
        const Grid g = size_grid(grid_rule(cd), axis_of_lane(lo), axis_of_lane(hi), ok);
        if (lane == 0) {
            *out = g;
            *s_ok = ok ? 1 : 0;
        }
    }
    __syncthreads();
    return *s_ok != 0;
}

// u . (T - p x F) for the wrench S = (F, T) and the joint axis u through p
__device__ __forceinline__ double axis_torque(const double4 &u, const double4 &p, const double *S)
{
    const double mx = S[3] - (p.y * S[2] - p.z * S[1]);
    const double my = S[4] - (p.z * S[0] - p.x * S[2]);
    const double mz = S[5] - (p.x * S[1] - p.y * S[0]);
    return u.x * mx + u.y * my + u.z * mz;
}
template <typename Chain>
__device__ __forceinline__ double joint_torque(const Chain *cd, int j, const double *S)
{
    return axis_torque(cd->jcur[2 * j], cd->jcur[2 * j + 1], S);
}

// Four sums over the wave, each as a tree of neighbours, ((v0 + v1) + (v2 +
// v3)) + ..., in lane 0.  The first two levels leave sum k in the lanes l with
// l mod 4 = k: 40 instructions in place of 104 for four sums in all lanes.
__device__ __forceinline__ void wave_tree_sum4(double *v)
{
    static_assert(WPART == 10, "four sums behind the wrench");
    const bool odd = threadIdx.x & 1, up = threadIdx.x & 2;
    const double a = (odd ? v[1] : v[0]) + dpp<DPP_QUAD_XOR1>(odd ? v[0] : v[1]);
    const double b = (odd ? v[3] : v[2]) + dpp<DPP_QUAD_XOR1>(odd ? v[2] : v[3]);
    double z = (up ? b : a) + dpp<DPP_QUAD_XOR2>(up ? a : b);
    z += __hiloint2double(from_xor4(__double2hiint(z)), from_xor4(__double2loint(z)));
    z += dpp<DPP_ROW_ROR + 8>(z);
    z = both_rows<false>(z) + both_rows<true>(z);
    z = both_halves<false>(z) + both_halves<true>(z);
    v[0] = z;
    v[1] = dpp<DPP_WAVE_SHL1>(z);
    v[2] = dpp<DPP_WAVE_SHL1>(v[1]);
    v[3] = dpp<DPP_WAVE_SHL1>(v[2]);
}

// Wrench (F, r x F), energies and failure flag of atom a at r (zeros past the
// chain's end), in two parts: the loads, and what is made of them.
struct AtomForce {
    double4 f, r, e;
    long long c[3];
};
template <typename Chain> __device__ __forceinline__ AtomForce load_force(const Chain *cd, int a)
{
    return {cd->f_pair[a], cd->r[a], cd->e_atom[a], {cd->f_cav[3 * a], cd->f_cav[3 * a + 1], cd->f_cav[3 * a + 2]}};
}
__device__ __forceinline__ void wrench_of(const AtomForce &in, bool valid, double4 &r, double (&v)[WPART])
{
#pragma unroll
    for (int k = 0; k < WPART; ++k) v[k] = 0.0;
    r = make_double4(0, 0, 0, 0);
    if (valid) {
        const double inv_fix = 1.0 / FIX_SCALE;
        const double Fx = in.f.x + (double)in.c[0] * inv_fix;
        const double Fy = in.f.y + (double)in.c[1] * inv_fix;
        const double Fz = in.f.z + (double)in.c[2] * inv_fix;
        r = in.r;
        v[0] = Fx; v[1] = Fy; v[2] = Fz;
        v[3] = r.y * Fz - r.z * Fy; v[4] = r.z * Fx - r.x * Fz; v[5] = r.x * Fy - r.y * Fx;
        v[6] = in.e.x; v[7] = in.e.y; v[8] = in.e.z;
        v[9] = (isfinite(Fx) && isfinite(Fy) && isfinite(Fz)) ? 0.0 : 1.0;
    }
}

// Over the wave: entries 0-5 (the wrench) become the inclusive suffix, this
// atom and every later one; entries 6-9 (energies, flag) in lane 0 the sum, in
// the order in which lane 0 of such a suffix adds.
__device__ __forceinline__ void wave_suffix(double (&S)[WPART])
{
    const int lane = threadIdx.x & (WAVE - 1);
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        double y[6];
#pragma unroll
        for (int k = 0; k < 6; ++k) y[k] = from_above(S[k], d);
        if (lane + d < WAVE) {
            masked_branch();
#pragma unroll
            for (int k = 0; k < 6; ++k) S[k] += y[k];
        }
    }
    wave_tree_sum4(S + 6);
}

// Adds to the suffix S of wave w the wrench of the W waves of its block after it;
// rows: the sums of the block's waves.  Lane k adds up component k, and all
// lanes take the six from there (33 instructions in place of 100, and three LDS
// reads in place of nine).
template <int W, typename Rows> __device__ __forceinline__ void add_later_waves(double (&S)[WPART], Rows rows, int w)
{
    const int lane = threadIdx.x & (WAVE - 1);
    double later = 0.0;
#pragma unroll
    for (int i = 1; i < W; ++i) {
        const double t = rows[i][min(lane, 5)];
        later = i > w ? later + t : later;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) S[k] += lane_value(later, k);
}

// Side-chain torque of the residue whose CB is atom a at r: the whole torque,
// over HB1..HB3 (atoms a+1 .. a+3), about the CA->CB axis through CA.
template <typename Chain>
__device__ __forceinline__ double chi_torque(const Chain *cd, int a, const double4 &r)
{
    const double inv_fix = 1.0 / FIX_SCALE;
    const double4 ca = cd->r[a - 2];
    double ux = r.x - ca.x, uy = r.y - ca.y, uz = r.z - ca.z;
    const double inv = 1.0 / sqrt(ux * ux + uy * uy + uz * uz);
    ux *= inv; uy *= inv; uz *= inv;
    double t = 0.0;
    for (int h = 1; h <= 3; ++h) {
        const int b = a + h;
        const double4 fp = cd->f_pair[b], rb = cd->r[b];
        const double Fx = fp.x + (double)cd->f_cav[3 * b] * inv_fix;
        const double Fy = fp.y + (double)cd->f_cav[3 * b + 1] * inv_fix;
        const double Fz = fp.z + (double)cd->f_cav[3 * b + 2] * inv_fix;
        const double dx = rb.x - ca.x, dy = rb.y - ca.y, dz = rb.z - ca.z;
        t += ux * (dy * Fz - dz * Fy) + uy * (dz * Fx - dx * Fz) + uz * (dx * Fy - dy * Fx);
    }
    return t;
}

// The compliance step of eq KCM_07 for the largest torque tm: dtheta = scale tau.
template <typename Chain>
__device__ __forceinline__ double step_scale(const Chain *cd, double tm)
{
    const double kappa = cd->kappa, smax = cd->max_step;
    if (cd->step_rule == 1) return tm > 0.0 ? smax / tm : 0.0;
    if (cd->step_rule == 2) return kappa;
    return (kappa * tm > smax) ? smax / tm : kappa;
}
__device__ __forceinline__ double stepped_angle(double th, double d)
{
    double t = th + d;
    if (t > PI_D) t -= 2.0 * PI_D;
    if (t <= -PI_D) t += 2.0 * PI_D;
    return t;
}

// ---------------------------------------------------------------------------
// k_tau: joint torques of the pending forces, one thread per joint
// ---------------------------------------------------------------------------
// k_wrench left in tau[j] the part of tau_j from the atoms of the workgroup
// that holds j's first downstream atom, and in wrench_part[b] the wrench sum
// (F, r x F) of atom workgroup b.  The rest comes from every later workgroup
// (the row scan of eq 04_9): tau_j += u_j . (T_later - p_j x F_later), eqs
// KCM_01-KCM_06.
__global__ __launch_bounds__(JOINT_BLOCK) void k_tau(Batch bt)
{
    const Owner own = owner_of(bt, bt.jblk_chain, bt.jblk_off, blockIdx.x);
    ChainStats *st = stats_of(own.cd);
    const ChainView view(own.cd), *cd = &view;
    __shared__ double s_red[(JOINT_BLOCK / WAVE) * 6];
    __shared__ double s_max[JOINT_BLOCK / WAVE];
    __shared__ int s_bad[JOINT_BLOCK / WAVE];
    __shared__ double s_S[8][6];
    const int jb = blockIdx.x - own.first;
    const int tid = threadIdx.x;
    const int J = cd->n_joints, n = cd->n_atoms;
    // the blocks of side-chain joints come last; k_wrench left each chi torque whole
    const bool chi = jb >= cd->n_bb_blocks;
    const int j = chi ? J + (jb - cd->n_bb_blocks) * JOINT_BLOCK + tid : jb * JOINT_BLOCK + tid;
    const int end = chi ? J + cd->n_chi : J, jc = min(j, end - 1), ja = min(jc, J - 1);
    double t = cd->tau[jc];
    const int moves = cd->mask[jc];
    const double4 u = cd->jcur[2 * ja], p = cd->jcur[2 * ja + 1];
    const int nblk = (n + ATOM_BLOCK - 1) / ATOM_BLOCK;
    const auto part = cd->wrench_part;
    // the joints of this workgroup take their later-workgroup wrench after
    // atom workgroups blo..bhi (at most 6 of them)
    const int jlo = min(jb * JOINT_BLOCK, J - 1), jhi = min(J, jlo + JOINT_BLOCK) - 1;
    const int blo = first_atom_of_joint(jlo) / ATOM_BLOCK, bhi = first_atom_of_joint(jhi) / ATOM_BLOCK;
    __shared__ double s_P[8][6];
    const double P = part[WPART * min(blo + tid / 6, nblk - 1) + tid % 6];
    double v[6] = {0, 0, 0, 0, 0, 0}, E[4] = {0, 0, 0, 0};
    if (!chi)
        for (int b = bhi + 1 + tid; b < nblk; b += JOINT_BLOCK)
#pragma unroll
            for (int k = 0; k < 6; ++k) v[k] += part[WPART * b + k];
    if (jb == 0)
        for (int b = tid; b < nblk; b += JOINT_BLOCK)
#pragma unroll
            for (int k = 0; k < 4; ++k) E[k] += part[WPART * b + 6 + k];
    loaded(t, moves, u, p, P, v[0], v[1], v[2], v[3], v[4], v[5], E[0], E[1], E[2], E[3]);
    if (!st->active || !st->pending_post) return;
    double tabs = 0.0;
    bool bad = false;
    if (!chi) {
        if (tid < 6 * (bhi - blo + 1)) s_P[tid / 6][tid % 6] = P;
        block_sum<6>(v, s_red);
        if (tid < 6) {
            // suffix over the touched workgroups, one wrench component per thread
            double x = v[tid];
            for (int b = bhi; b >= blo; --b) {
                s_S[b - blo][tid] = x;
                x += s_P[b - blo][tid];
            }
        }
        lds_barrier();
        if (j < end) {
            t += axis_torque(u, p, s_S[first_atom_of_joint(j) / ATOM_BLOCK - blo]);
            cd->tau[j] = t;
        }
    }
    if (j < end) {
        bad = !isfinite(t);
        if (moves) tabs = fabs(t);
    }
    const double tmax = block_max_any(tabs, bad, s_max, s_bad);
    if (tid == 0) {
        cd->tmax_part[jb] = tmax;
        cd->bad_part[jb] = bad ? 1 : 0;
    }
    if (jb == 0) {
        // energies and the non-finite force flag of the pending forces
        block_sum<4>(E, s_red);
        if (tid == 0) {
            st->e_elec = E[0];
            st->e_vdw = E[1];
            st->e_cav = E[2];
            st->post_bad = E[3] > 0.0 ? 1 : 0;
        }
    }
}

// ---------------------------------------------------------------------------
// k_stepfk: compliance step of the pending forces (eq KCM_07), then the
// kinematics of the new angles inside each joint block (eqs kin_02-kin_04,
// r1): xform_loc[j] = T_{jlo} o ... o T_j by an ordered scan, and the block
// product in blk_xf.  k_place composes the products of earlier blocks in
// front (prefix computation, item 1 of Sec. 3.5).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(JOINT_BLOCK) void k_stepfk(Batch bt, int mode)
{
    const Owner own = owner_of(bt, bt.jblk_chain, bt.jblk_off, blockIdx.x);
    ChainStats *st = stats_of(own.cd);
    const ChainView view(own.cd), *cd = &view;
    __shared__ double s_red[JOINT_BLOCK / WAVE];
    __shared__ int s_bad[JOINT_BLOCK / WAVE];
    __shared__ double s_x[JOINT_BLOCK / WAVE][12];
    const int jb = blockIdx.x - own.first;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
    const int J = cd->n_joints;
    // backbone blocks first; the blocks after them hold the side-chain joints,
    // which step with the others but are not part of the chain's scan
    const bool chi_block = jb >= cd->n_bb_blocks;
    const int j = chi_block ? J + (jb - cd->n_bb_blocks) * JOINT_BLOCK + tid : jb * JOINT_BLOCK + tid;
    const bool valid = chi_block ? j < J + cd->n_chi : j < J;
    const int jv = min(j, (chi_block ? J + cd->n_chi : J) - 1), ja = min(jv, J - 1);
    double th = cd->theta[jv];
    const double tau = cd->tau[jv];
    const int moves = cd->mask[jv];
    const double4 u0 = cd->joint0[2 * ja], p0 = cd->joint0[2 * ja + 1];
    const int nb = cd->n_bb_blocks + (cd->n_chi + JOINT_BLOCK - 1) / JOINT_BLOCK;
    double tm = 0.0;
    int bad_parts = 0;
    for (int b = tid; b < nb; b += JOINT_BLOCK) {
        tm = fmax(tm, cd->tmax_part[b]);
        bad_parts |= cd->bad_part[b];
    }
    loaded(th, tau, moves, u0, p0, tm, bad_parts);
    if (!st->active) return;
    if (mode == MODE_BOOT && (chi_block || !st->need_grid)) return;
    const bool lead = jb == 0 && tid == 0;

    if (mode != MODE_BOOT && st->pending_post) {
        bool bad = bad_parts != 0;
        tm = block_max_any(tm, bad, s_red, s_bad);
        if (bad || st->post_bad) {
            if (lead) {
                st->status = -4;
                st->run = 0;
            }
            return;
        }
        const double scale = step_scale(cd, tm);
        if (valid) {
            const double d = moves ? scale * tau : 0.0;
            cd->dtheta[j] = d;
            th = stepped_angle(th, d);
            cd->theta[j] = th;
        }
        if (lead) {
            // max |dtheta| over the moving joints is scale * max |tau| exactly
            const double mxd = scale * tm;
            st->max_tau = tm;
            st->max_dtheta = mxd;
            st->iterations += 1;
            if (st->nbr_overflow) st->status = -6;
            int go = 1;
            if (st->tol > 0.0 && mxd < st->tol) {
                st->converged = 1;
                go = 0;
            }
            if (st->iterations >= st->iter_limit) go = 0;
            st->run = go;
        }
    } else if (lead && mode != MODE_BOOT) {
        st->run = 1;
    }
    if (mode == MODE_FINAL || chi_block) return;

    Xf x = xf_identity();
    if (valid) x = joint_xf_of(u0, p0, th);
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        Xf y = xf_from_below(x, d);
        if (lane >= d) {
            masked_branch();
            x = xf_mul(y, x);
        }
    }
    if (lane == WAVE - 1) xf_store(s_x[w], x);
    lds_barrier();
    if (w > 0) {
        Xf pre = xf_load(s_x[0]);
        for (int i = 1; i < w; ++i) pre = xf_mul(pre, xf_load(s_x[i]));
        x = xf_mul(pre, x);
    }
    if (valid) xf_store(cd->xform_loc + 12 * j, x);
    if (tid == min(J - jb * JOINT_BLOCK, JOINT_BLOCK) - 1) xf_store(cd->blk_xf + 12 * jb, x);
}

// Position of atom a with zero position q under its link transform L.
template <typename Chain>
__device__ __forceinline__ double4 placed_atom(const Chain *cd, int a, double4 q, const double *L)
{
    const int res = a / APR, slot = a - res * APR;
    if (cd->n_chi && slot >= 5 && slot <= 7) {
        // side-chain joint chi of the residue (dihedral N-CA-CB-HB1, 60
        // degrees in the zero position): HB1..HB3 turn about CA->CB, here
        // in the zero-position frame before the link transform
        const double4 ca = cd->r0[res * APR + 2], cb = cd->r0[res * APR + 4];
        double ux = cb.x - ca.x, uy = cb.y - ca.y, uz = cb.z - ca.z;
        const double inv = 1.0 / sqrt(ux * ux + uy * uy + uz * uz);
        ux *= inv; uy *= inv; uz *= inv;
        double sn, cs;
        sincos(cd->theta[cd->n_joints + res] - PI_D / 3.0, &sn, &cs);
        const double vx = q.x - cb.x, vy = q.y - cb.y, vz = q.z - cb.z;
        const double dot = ux * vx + uy * vy + uz * vz;
        const double wx = uy * vz - uz * vy, wy = uz * vx - ux * vz, wz = ux * vy - uy * vx;
        q.x = cb.x + vx * cs + wx * sn + ux * dot * (1.0 - cs);
        q.y = cb.y + vy * cs + wy * sn + uy * dot * (1.0 - cs);
        q.z = cb.z + vz * cs + wz * sn + uz * dot * (1.0 - cs);
    }
    double4 r;
    r.x = L[0] * q.x + L[1] * q.y + L[2] * q.z + L[9];
    r.y = L[3] * q.x + L[4] * q.y + L[5] * q.z + L[10];
    r.z = L[6] * q.x + L[7] * q.y + L[8] * q.z + L[11];
    r.w = 0.0;
    return r;
}

// ---------------------------------------------------------------------------
// k_place: link transforms of this workgroup's links, positions
// r_a = G_link(a) r0_a, cell keys and counts, bounding box
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(ATOM_BLOCK) void k_place(Batch bt, int mode)
{
    const Owner own = owner_of(bt, bt.blk_chain, bt.blk_off, blockIdx.x);
    ChainStats *st = stats_of(own.cd);
    const ChainView view(own.cd), *cd = &view;
    const int lb = blockIdx.x - own.first;
    __shared__ double s_G[LINKS_PER_BLOCK][12];
    __shared__ double s_c[2][12];
    __shared__ double s_bb[ATOM_BLOCK / WAVE][6];
    __shared__ int s_bad[ATOM_BLOCK / WAVE];
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
    const int n = cd->n_atoms;
    const int a0 = lb * ATOM_BLOCK, a1 = min(n, a0 + ATOM_BLOCK) - 1;
    const int l_lo = link_of_atom(a0), l_hi = link_of_atom(a1);
    // link l (>= 1) needs the product of the joint blocks before joint l-1
    const int jb_lo = (max(l_lo, 1) - 1) / JOINT_BLOCK, jb_hi = (max(l_hi, 1) - 1) / JOINT_BLOCK;
    // zero position of the thread's atom, transform inside its block and joint of its link
    const int a = a0 + tid, nL = l_hi - l_lo + 1, jl = max(l_lo + min(tid, nL - 1), 1) - 1;
    const double4 r0 = cd->r0[min(a, n - 1)];
    const Xf loc = xf_load(cd->xform_loc + 12 * jl);
    const double4 u0 = cd->joint0[2 * jl], p0 = cd->joint0[2 * jl + 1];
    static_assert(LINKS_PER_BLOCK <= ATOM_BLOCK, "a thread for each link");
    if (tid < nL) xf_store(s_G[tid], loc);  // there until it is used: registers decide how many waves fit
    loaded(r0, u0, p0);
    // the step and torque kernels of this iteration have consumed the pending forces
    if (mode == MODE_ITER && lb == 0 && tid == 0) st->pending_post = 0;
    if (mode == MODE_BOOT ? !(st->active && st->need_grid) : !running(st)) return;
    if (w == 0) {
        Xf acc = xf_identity();
        for (int base = 0; base < jb_hi; base += WAVE) {
            Xf x = (base + lane < jb_hi) ? xf_load(cd->blk_xf + 12 * (base + lane)) : xf_identity();
#pragma unroll
            for (int d = 1; d < WAVE; d <<= 1) {
                Xf y = xf_from_below(x, d);
                if (lane >= d) {
                    masked_branch();
                    x = xf_mul(y, x);
                }
            }
            if (base > 0) x = xf_mul(acc, x);
            if (base + lane == jb_lo - 1) xf_store(s_c[0], x);
            if (base + lane == jb_hi - 1) xf_store(s_c[1], x);
            acc = xf_shfl_idx(x, WAVE - 1);
        }
        if (lane == 0) {
            if (jb_lo == 0) xf_store(s_c[0], xf_identity());
            if (jb_hi == 0) xf_store(s_c[1], xf_identity());
        }
    }
    lds_barrier();
    if (tid < nL) {
        const int l = l_lo + tid;
        Xf G = xf_identity();
        if (l > 0) {
            masked_branch();
            G = xf_mul(xf_load(s_c[jl / JOINT_BLOCK == jb_lo ? 0 : 1]), xf_load(s_G[tid]));
        }
        xf_store(s_G[tid], G);
        const int fa = first_atom_of_link(l);
        if (l > 0 && fa >= a0 && fa <= a1) {
            masked_branch();
            fk_emit(G, jl, u0, p0, cd->jcur);
        }
    }
    lds_barrier();

    double lo[3] = {DBL_MAX, DBL_MAX, DBL_MAX}, hi[3] = {-DBL_MAX, -DBL_MAX, -DBL_MAX};
    bool fin = true;
    if (a <= a1) {
        const double4 r = placed_atom(cd, a, r0, s_G[link_of_atom(a) - l_lo]);
        cd->r[a] = r;
        fin = isfinite(r.x) && isfinite(r.y) && isfinite(r.z);
        if (mode == MODE_ITER) {
            cd->f_cav[3 * a] = 0;
            cd->f_cav[3 * a + 1] = 0;
            cd->f_cav[3 * a + 2] = 0;
        }
        lo[0] = r.x; lo[1] = r.y; lo[2] = r.z;
        hi[0] = r.x; hi[1] = r.y; hi[2] = r.z;
    }
    wave_box(lo, hi);
    const bool bad_w = __any(!fin);
    if (lane == 0) {
        for (int k = 0; k < 3; ++k) { s_bb[w][k] = lo[k]; s_bb[w][3 + k] = hi[k]; }
        s_bad[w] = bad_w ? 1 : 0;
    }
    lds_barrier();
    if (tid < 6) {
        const int k = tid;
        double v = s_bb[0][k];
        int bad = s_bad[0];
        for (int i = 1; i < ATOM_BLOCK / WAVE; ++i) {
            v = (k < 3) ? fmin(v, s_bb[i][k]) : fmax(v, s_bb[i][k]);
            bad |= s_bad[i];
        }
        cd->bbox_part[6 * lb + k] = bad ? NAN : v;
    }
}

// ---------------------------------------------------------------------------
// k_grid and k_cellkey: this iteration's grid of Sec. 3.2, sized from the
// bounding box of the positions just placed plus a margin, then every atom's
// cell key and the cell counts.  The grid is a function of the current
// conformation alone, so a chain rebuilt from saved angles continues exactly
// as the original.  Two launch forms with the same grid and keys: for large
// batches one wave per chain sizes the grid (k_grid) and the key workgroups
// read it; for small ones, where a launch costs more than the redundant work,
// wave 0 of every key workgroup sizes it and the first one stores it.
// ---------------------------------------------------------------------------
// the grid from the chain's bounding-box partials (one wave)
__device__ __forceinline__ Grid wave_grid(const ChainView *cd, bool *ok)
{
    const int lane = (int)threadIdx.x & (WAVE - 1), nblk = (cd->n_atoms + ATOM_BLOCK - 1) / ATOM_BLOCK;
    double lo[3] = {DBL_MAX, DBL_MAX, DBL_MAX}, hi[3] = {-DBL_MAX, -DBL_MAX, -DBL_MAX};
    bool fin = true;
    for (int b = lane; b < nblk; b += WAVE)
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const double l = cd->bbox_part[6 * b + k], h = cd->bbox_part[6 * b + 3 + k];
            fin = fin && isfinite(l) && isfinite(h);
            lo[k] = fmin(lo[k], l);
            hi[k] = fmax(hi[k], h);
        }
    wave_box(lo, hi);
    *ok = fin;
    return size_grid(grid_rule(cd), axis_of_lane(lo), axis_of_lane(hi), *ok);
}

__device__ __forceinline__ void store_grid(Grid *out, ChainStats *st, const Grid &g, bool ok)
{
    if (ok) {
        *out = g;
    } else {
        st->status = -4;
        st->grid_bad = 1;
    }
}

__global__ __launch_bounds__(WAVE) void k_grid(Batch bt)
{
    const ChainDev *dev = bt.n_chains == 1 ? bt.only : bt.table[blockIdx.x];
    ChainStats *st = stats_of(dev);
    const ChainView view(dev);
    if (!running(st)) return;
    bool ok;
    const Grid g = wave_grid(&view, &ok);
    if (threadIdx.x == 0) store_grid(grid_of(dev), st, g, ok);
}

template <bool OWN_GRID>
__global__ __launch_bounds__(ATOM_BLOCK) void k_cellkey(Batch bt)
{
    const Owner own = owner_of(bt, bt.blk_chain, bt.blk_off, blockIdx.x);
    ChainStats *st = stats_of(own.cd);
    const ChainView view(own.cd), *cd = &view;
    const int lb = blockIdx.x - own.first, a = lb * ATOM_BLOCK + threadIdx.x;
    const bool valid = a < cd->n_atoms;
    const double4 r = cd->r[min(a, cd->n_atoms - 1)];
    loaded(r);
    // with OWN_GRID, grid_bad is set by this kernel: a workgroup that sees it
    // set by the first one would have found the same failure itself
    if (!running(st)) return;
    __shared__ int s_ok;
    __shared__ Grid s_g;
    // Atoms of the workgroup that share a cell take one count atomic between
    // them: an LDS table (open addressing on the key, twice as many slots as
    // atoms, so a probe always ends) gives each atom its rank among them, the
    // first adds their number to the cell's count, and each atom's place among
    // the cell's arrivals is the returned base plus its rank.
    constexpr int HSLOTS = 2 * ATOM_BLOCK;
    __shared__ int s_hkey[HSLOTS], s_hcnt[HSLOTS], s_hbase[HSLOTS];
    for (int h = threadIdx.x; h < HSLOTS; h += ATOM_BLOCK) {
        s_hkey[h] = -1;
        s_hcnt[h] = 0;
    }
    if (OWN_GRID) {
        if (threadIdx.x < WAVE) {
            bool ok;
            const Grid g = wave_grid(cd, &ok);
            if (threadIdx.x == 0) {
                s_g = g;
                s_ok = ok ? 1 : 0;
                if (lb == 0) store_grid(grid_of(own.cd), st, g, ok);
            }
        }
    } else if (threadIdx.x == 0) {
        s_g = *grid_of(own.cd);
    }
    lds_barrier();
    if (OWN_GRID && !s_ok) return;
    int key = 0, slot = 0, rank = 0;
    if (valid) {
        key = cell_of(s_g, r);
        cd->cell_key[a] = key;
        slot = (int)(((unsigned)key * 2654435761u) >> 23) & (HSLOTS - 1);
        for (;;) {
            const int prev = atomicCAS(&s_hkey[slot], -1, key);
            if (prev == -1 || prev == key) break;
            slot = (slot + 1) & (HSLOTS - 1);
        }
        rank = atomicAdd(&s_hcnt[slot], 1);
    }
    lds_barrier();
    if (valid && rank == 0) s_hbase[slot] = atomicAdd(&own.cd->cell_count[key], s_hcnt[slot]);
    lds_barrier();
    // kept for the scatter in the sorted-index array (free until the rank
    // kernel fills it)
    if (valid) cd->s_idx[a] = s_hbase[slot] + rank;
}

// ---------------------------------------------------------------------------
// k_gridboot: first grid of a chain whose conformation has no grid yet
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(CHAIN_THREADS) void k_gridboot(Batch bt)
{
    ChainDev *cd = bt.n_chains == 1 ? bt.only : bt.table[blockIdx.x];
    ChainStats *st = stats_of(cd);
    if (!st->active || !st->need_grid) return;
    __shared__ double s_red[CHAIN_THREADS / WAVE * 6];
    __shared__ int s_ok;
    const bool ok = grid_from_parts(cd, grid_of(cd), s_red, &s_ok);
    if (threadIdx.x == 0) {
        st->need_grid = 0;
        if (!ok) {
            st->status = -4;
            st->active = 0;
            st->run = 0;
        }
    }
}

// k_finish: the call's last post phase is applied; the chain's state for the
// next call is its run flag.
__global__ void k_finish(Batch bt)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= bt.n_chains) return;
    ChainStats *st = stats_of(bt.table[c]);
    st->pending_post = 0;
    st->active = running(st);
}

// Stores seq to a flag in pinned host memory once every store of the workgroup
// before it has reached the host (one workgroup).
__device__ __forceinline__ void signal_host(unsigned *flag, unsigned seq)
{
    __threadfence_system();
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(flag, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// k_stats_gather: the records of every chain of the batch into one array, so
// that the host reads them back at once.  With a flag one workgroup does it all.
__global__ __launch_bounds__(1024) void k_stats_gather(Batch bt, ChainStats *__restrict__ out, unsigned *flag, unsigned seq)
{
    constexpr int W = sizeof(ChainStats) / sizeof(double);
    static_assert(W * sizeof(double) == sizeof(ChainStats), "records are whole doubles");
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < (int64_t)W * bt.n_chains; i += (int64_t)gridDim.x * blockDim.x)
        reinterpret_cast<double *>(out)[i] = reinterpret_cast<const double *>(stats_of(bt.table[i / W]))[i % W];
    if (flag) signal_host(flag, seq);
}

// k_box_read: a host read's values into pinned memory, then the flag of each
// workgroup's share.  All parts are one run of values, a thread for each where
// they are few, so that the kernel waits for one round of loads and not for one
// per part, and no wave without a value has a store to wait for (the angles of
// a chain of 20 residues: 2.4 us, 2.8 with four waves and part after part).
__global__ __launch_bounds__(1024) void k_box_read(BoxRead what, double *__restrict__ out, unsigned *flags, unsigned seq)
{
    int total = 0;
#pragma unroll
    for (int k = 0; k < BOX_PARTS; ++k) total += (int)what.n[k];
#pragma unroll 4
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
        const double *src = what.src[0];
        const long long *cav = what.f_cav[0];
        bool atoms = what.atoms[0];
        int first = 0, j = i;
#pragma unroll
        for (int k = 1; k < BOX_PARTS; ++k) {
            first += (int)what.n[k - 1];
            if (i >= first) {
                src = what.src[k];
                cav = what.f_cav[k];
                atoms = what.atoms[k];
                j = i - first;
            }
        }
        double v = glob(src)[atoms ? j + j / 3 : j];  // x, y, z of every four
        if (cav) v += (double)glob(cav)[j] / FIX_SCALE;
        out[i] = v;
    }
    signal_host(flags + blockIdx.x, seq);
}

// k_fold_control: FOLD_BEGIN keeps the chain's own stopping rule
// (kcm_set_limits) aside and arms every chain for a fold of at most max_iter
// iterations that stops below tol (a chain with a failure status stays
// stopped); FOLD_END puts the chain's own rule back and leaves every chain
// steppable again unless it converged, failed or reached its own limit.
__global__ void k_fold_control(Batch bt, int mode, double tol, int64_t max_iter)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= bt.n_chains) return;
    ChainStats *st = stats_of(bt.table[c]);
    if (mode == FOLD_BEGIN) {
        const int go = st->status == 0 && max_iter > 0 ? 1 : 0;
        st->saved_tol = st->tol;
        st->saved_limit = st->iter_limit;
        st->tol = tol;
        st->iter_limit = st->iterations + max_iter;
        st->converged = 0;
        st->active = go;
        st->run = go;
    } else {
        st->tol = st->saved_tol;
        st->iter_limit = st->saved_limit;
        const int again = st->status == 0 && !st->converged && st->iterations < st->iter_limit ? 1 : 0;
        st->active = again;
        st->run = again;
    }
}

// ---------------------------------------------------------------------------
// Monte Carlo minimization over the descent (the hybrid of Monte Carlo
// sampling and steepest descent among the search improvements of Sec. 4, in
// the form of Li and Scheraga): perturb the accepted angles, descend, keep the
// descended state by the Metropolis rule on its energy.  Three small kernels
// around the ordinary iterations; the random numbers are inputs.
// ---------------------------------------------------------------------------
// joint j of workgroup jb of a chain's joint blocks (backbone blocks, then
// side-chain blocks); false past the end
__device__ __forceinline__ bool joint_of_block(const ChainDev *cd, int jb, int tid, int *j)
{
    if (jb >= cd->n_bb_blocks) {
        const int jc = (jb - cd->n_bb_blocks) * JOINT_BLOCK + tid;
        *j = cd->n_joints + jc;
        return jc < cd->n_chi;
    }
    *j = jb * JOINT_BLOCK + tid;
    return *j < cd->n_joints;
}

// angle into (-pi, pi]; an angle already inside comes back unchanged
__device__ __forceinline__ double wrap_angle(double t)
{
    t -= 2.0 * PI_D * floor((t + PI_D) / (2.0 * PI_D));
    return t <= -PI_D ? t + 2.0 * PI_D : t;
}

// MC_RESET: the chain re-boots from its current angles (positions, grid),
// with no convergence test or iteration limit, so that every descent runs its
// full length.  MC_PROPOSE: angles = wrap(accepted + delta of this trial) on
// the free joints, then the same re-boot.  A chain with a failure status is
// left alone.
__global__ __launch_bounds__(JOINT_BLOCK) void k_mc_propose(Batch bt, int mode, const double *__restrict__ delta,
                                                             const int64_t *__restrict__ delta_off, int trial)
{
    const Owner own = owner_of(bt, bt.jblk_chain, bt.jblk_off, blockIdx.x);
    ChainDev *cd = own.cd;
    ChainStats *st = stats_of(cd);
    if (st->status != 0) return;
    const int jb = blockIdx.x - own.first;
    if (jb == 0 && threadIdx.x == 0) {
        st->need_grid = 1;
        st->pending_post = 0;
        st->post_bad = 0;
        st->converged = 0;
        st->tol = 0.0;
        st->iter_limit = INT64_MAX;
        st->run = 1;
        st->active = 1;
    }
    int j;
    if (mode != MC_PROPOSE || !joint_of_block(cd, jb, threadIdx.x, &j)) return;
    const int Jt = cd->n_joints + cd->n_chi;
    const double a = cd->mc_theta[j];
    cd->theta[j] = cd->mask[j] ? wrap_angle(a + delta[delta_off[own.chain] + (int64_t)trial * Jt + j]) : a;
}

// One thread per chain, after the torque kernel has reduced the energies of
// the last evaluation.  MC_INIT takes the state as the accepted and lowest
// one; MC_TRIAL accepts it when E <= E_acc or u < exp(-(E - E_acc)/kT).  The
// pending step of the last evaluation is discarded either way.
__global__ void k_mc_decide(Batch bt, int mode, const double *__restrict__ u, int n_trials, int trial, double kT)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= bt.n_chains) return;
    const ChainDev *cd = bt.table[c];
    ChainStats *st = stats_of(cd);
    // the energy of the chain's terms (bits 1 Coulomb, 2 Lennard-Jones, 4 solvation)
    double e = 0.0;
    if (cd->terms & 1) e += st->e_elec;
    if (cd->terms & 2) e += st->e_vdw;
    if (cd->terms & 4) e += st->e_cav;
    if (st->status == 0 && (st->post_bad || !isfinite(e))) st->status = -4;
    const int ok = st->status == 0;
    int acc = 0, best = 0;
    if (mode == MC_INIT) {
        // taken even after a failure, so that the accepted angles are defined
        acc = best = 1;
        st->mc_e_start = st->mc_e_acc = st->mc_e_best = e;
        st->mc_trials = st->mc_accepted = 0;
    } else if (ok) {
        const double de = e - st->mc_e_acc;
        acc = de <= 0.0 || (kT > 0.0 && u[(int64_t)c * n_trials + trial] < exp(-de / kT));
        best = e < st->mc_e_best;
        if (acc) st->mc_e_acc = e;
        if (best) st->mc_e_best = e;
        st->mc_trials += 1;
        st->mc_accepted += acc;
    }
    st->mc_acc = acc;
    st->mc_best = best;
    st->pending_post = 0;
    st->need_grid = 1;
    st->active = ok;
    st->run = ok;
}

// Joint blocks: the lowest and accepted angles take the trial's angles as
// decided; a rejected trial returns the chain to the accepted angles.
__global__ __launch_bounds__(JOINT_BLOCK) void k_mc_apply(Batch bt)
{
    const Owner own = owner_of(bt, bt.jblk_chain, bt.jblk_off, blockIdx.x);
    ChainDev *cd = own.cd;
    const ChainStats *st = stats_of(cd);
    int j;
    if (!joint_of_block(cd, blockIdx.x - own.first, threadIdx.x, &j)) return;
    const int Jt = cd->n_joints + cd->n_chi;
    const double p = cd->theta[j];
    if (st->mc_best) cd->mc_theta[Jt + j] = p;
    if (st->mc_acc) cd->mc_theta[j] = p;
    else cd->theta[j] = cd->mc_theta[j];
}

// New angles for every chain of the batch from one device array (chain c's
// J_c angles at theta_off[c]), wrapped into (-pi, pi]; each chain restarts
// like a freshly built one (flags cleared, positions and grid anew).
__global__ __launch_bounds__(JOINT_BLOCK) void k_set_theta(Batch bt, const double *__restrict__ theta,
                                                            const int64_t *__restrict__ theta_off)
{
    const Owner own = owner_of(bt, bt.jblk_chain, bt.jblk_off, blockIdx.x);
    ChainDev *cd = own.cd;
    const int jb = blockIdx.x - own.first;
    if (jb == 0 && threadIdx.x == 0) {
        ChainStats *st = stats_of(cd);
        st->converged = 0;
        st->status = 0;
        st->nbr_overflow = 0;
        st->need_grid = 1;
        st->pending_post = 0;
        st->post_bad = 0;
        st->grid_bad = 0;
        st->run = 1;
        st->active = 1;
    }
    int j;
    if (!joint_of_block(cd, jb, threadIdx.x, &j)) return;
    cd->theta[j] = wrap_angle(theta[theta_off[own.chain] + j]);
}

// ---------------------------------------------------------------------------
// cell list: exclusive scan of the counts, counting-sort scatter, stable
// order inside each cell, gather into cell order
// ---------------------------------------------------------------------------
// Chunk offsets of the chain's current grid, block-wide: s_off[b] = number of
// atoms in the cells of the chunks before chunk b, for b = 0 .. nb (s_off[nb]:
// all atoms).  The cell start of cell c is cell_local[c] + s_off[c / SCAN_CHUNK].
__device__ __forceinline__ void chunk_offsets(const ChainView *cd, int nc, int *s_off, int *s_int)
{
    const int nb = (nc + SCAN_CHUNK - 1) / SCAN_CHUNK;
    const int tid = threadIdx.x, per = (nb + blockDim.x - 1) / blockDim.x;
    int loc = 0;
    for (int k = 0; k < per; ++k) {
        const int b = tid * per + k;
        if (b < nb) loc += cd->scan_part[b];
    }
    int total = 0;
    int run = block_excl_scan(loc, s_int, &total);
    if (per == 1) {
        if (tid < nb) s_off[tid] = run;
    } else {
        for (int k = 0; k < per; ++k) {
            const int b = tid * per + k;
            if (b < nb) {
                s_off[b] = run;
                run += cd->scan_part[b];
            }
        }
    }
    if (tid == 0) s_off[nb] = total;
    lds_barrier();
}

// Parameters of an atom as the cell-ordered array s_p holds them: (q, R,
// sqrt(eps), R_off) in FP64, or, for a chain of the mixed form, the first three
// as the FP32 values its pair terms use in the first 16 bytes.  Either way
// R_off is the last double.
template <typename Chain>
__device__ __forceinline__ double4 sorted_param(const Chain *cd, double4 p)
{
    if (cd->precision == 1) {
        p.x = __hiloint2double(__float_as_int((float)p.y), __float_as_int((float)p.x));
        p.y = __hiloint2double(0, __float_as_int((float)p.z));
        p.z = 0.0;
    }
    return p;
}

// k_cellscan: one workgroup per chunk of SCAN_CHUNK cells of each chain's
// capacity (chunks past the current grid return at once): the exclusive scan
// of the counts inside the chunk, and the chunk's total.  Each thread takes
// four consecutive cells as one 16-byte load (the capacity is a multiple of
// 8 cells, so a load that starts inside the grid stays inside the array),
// scans them in registers, and the block scans the thread totals.  The chunk
// offsets are added by the scatter and rank kernels; k_rank writes the final
// starts.
__global__ __launch_bounds__(CHAIN_THREADS) void k_cellscan(Batch bt)
{
    static_assert(SCAN_CHUNK == 4 * CHAIN_THREADS, "four cells per thread");
    const Owner own = owner_of(bt, bt.scan_chain, bt.scan_off, blockIdx.x);
    const ChainView view(own.cd), *cd = &view;
    const int b = blockIdx.x - own.first, c0 = b * SCAN_CHUNK, i0 = 4 * (int)threadIdx.x;
    int4 v = *(const gptr<const int4>)(cd->cell_count + min(c0 + i0, cd->cap_cells - 4));
    loaded(v.x, v.y, v.z, v.w);
    const int nc = grid_of(own.cd)->n_cells;
    if (!running(stats_of(own.cd)) || c0 >= nc) return;
    __shared__ int s_int[CHAIN_THREADS / WAVE];
    const int m = min(SCAN_CHUNK, nc - c0);
    if (i0 >= m) v.x = 0;
    if (i0 + 1 >= m) v.y = 0;
    if (i0 + 2 >= m) v.z = 0;
    if (i0 + 3 >= m) v.w = 0;
    int total = 0;
    const int run = block_excl_scan(v.x + v.y + v.z + v.w, s_int, &total);
    const int4 o = make_int4(run, run + v.x, run + v.x + v.y, run + v.x + v.y + v.z);
    const auto local = cd->cell_local + c0 + i0;
    if (i0 + 3 < m) {
        *(gptr<int4>)local = o;
    } else if (i0 < m) {
        local[0] = o.x;
        if (i0 + 1 < m) local[1] = o.y;
        if (i0 + 2 < m) local[2] = o.z;
    }
    if (threadIdx.x == 0) cd->scan_part[b] = total;
}

// k_scatter and k_rank: one thread per atom; the dynamic LDS holds the chunk
// offsets (SCAN_MAX_CHUNKS + 1 ints at most).
__global__ __launch_bounds__(ATOM_BLOCK) void k_scatter(Batch bt)
{
    extern __shared__ int s_off[];
    __shared__ int s_int[ATOM_BLOCK / WAVE];
    const Owner own = owner_of(bt, bt.blk_chain, bt.blk_off, blockIdx.x);
    const ChainView view(own.cd), *cd = &view;
    const int a = (blockIdx.x - own.first) * ATOM_BLOCK + threadIdx.x, ac = min(a, cd->n_atoms - 1);
    const int key = cd->cell_key[ac], arrival = cd->s_idx[ac];
    loaded(key, arrival);
    const int nc = grid_of(own.cd)->n_cells;
    if (!running(stats_of(own.cd))) return;
    const int local = cd->cell_local[key];
    chunk_offsets(cd, nc, s_off, s_int);
    if (a < cd->n_atoms) cd->s_tmp[local + s_off[key / SCAN_CHUNK] + arrival] = a;
}

// The counting-sort scatter placed the atoms of a cell in the order of their
// count atomics; the stable slot is the number of atoms of the cell with a
// smaller index, so everything downstream is deterministic.  Gathers position
// and parameters into that slot; w holds the atom index in its low and the
// atom's residue in its high 32 bits (read as integers only).
__global__ __launch_bounds__(ATOM_BLOCK) void k_rank(Batch bt)
{
    extern __shared__ int s_off[];
    __shared__ int s_int[ATOM_BLOCK / WAVE];
    const Owner own = owner_of(bt, bt.blk_chain, bt.blk_off, blockIdx.x);
    const ChainView view(own.cd), *cd = &view;
    const int lb = blockIdx.x - own.first, nblk = (cd->n_atoms + ATOM_BLOCK - 1) / ATOM_BLOCK;
    const int a = lb * ATOM_BLOCK + threadIdx.x, ac = min(a, cd->n_atoms - 1);
    const int key = cd->cell_key[ac];
    const double4 r = cd->r[ac], ap = cd->aparam[ac];
    loaded(key, r, ap, ap.w);
    const int nc = grid_of(own.cd)->n_cells, nb = (nc + SCAN_CHUNK - 1) / SCAN_CHUNK;
    if (!running(stats_of(own.cd))) return;
    const int local = cd->cell_local[key], next = cd->cell_local[min(key + 1, nc - 1)];
    chunk_offsets(cd, nc, s_off, s_int);
    const int b = local + s_off[key / SCAN_CHUNK];
    const int e = key + 1 < nc ? next + s_off[(key + 1) / SCAN_CHUNK] : s_off[nb];
    // the cell's members four at a time, every load issued before any is
    // compared (indices clamped into the cell, which holds a itself, e > b)
    int pos = b;
    for (int s = b; s < e; s += 4) {
        int v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = cd->s_tmp[min(s + k, e - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) pos += (s + k < e && v[k] < a) ? 1 : 0;
    }
    if (a < cd->n_atoms) {
        cd->s_idx[pos] = a;
        cd->s_r[pos] = make_double4(r.x, r.y, r.z, __longlong_as_double((long long)a | ((long long)(a / APR) << 32)));
        cd->s_p[pos] = sorted_param(cd, ap);
        // the first atom of each cell returns its count to zero for the next iteration
        if (pos == b) cd->cell_count[key] = 0;
    }
    // the final cell starts (nc + 1 of them), a slice per workgroup of the
    // chain: four cells per thread per step, the loads issued before the stores
    // (indices clamped into the grid, which has at least one cell)
    const int per = (nc + 1 + nblk - 1) / nblk, i1 = min(nc + 1, (lb + 1) * per);
    for (int i = lb * per + (int)threadIdx.x; i < i1; i += 4 * ATOM_BLOCK) {
        int v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = cd->cell_local[min(i + k * ATOM_BLOCK, nc - 1)];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int j = i + k * ATOM_BLOCK;
            if (j < i1) cd->cell_start[j] = j < nc ? v[k] + s_off[j / SCAN_CHUNK] : s_off[nb];
        }
    }
}

// ---------------------------------------------------------------------------
// k_chain: everything of an iteration but the force kernel, one workgroup per
// chain, for calls of short or many chains (set_form in kcm_host.cpp)
// ---------------------------------------------------------------------------
// The same work as k_wrench, k_tau, k_stepfk, k_place, k_cellkey, k_cellscan,
// k_scatter and k_rank (and of k_gridboot and k_finish), with the same
// arithmetic in the same order -- scans and sums in blocks of 256 joints or
// atoms -- so a chain's results do not depend on which form a call takes.
// What those kernels hand over through memory and a launch boundary stays in
// LDS and registers here: link transforms, torques, cell counts (16 bits
// each: at most CHAIN_ATOMS atoms) and the scatter.  Order within a call:
// MODE_ITER applies the forces of the iteration before it, if they are
// pending, and prepares the force kernel's inputs; MODE_FINAL applies the last
// ones and ends the call; MODE_TAU leaves torques and energies only.
// The conditions that end the kernel early are the same for all threads, so
// every barrier is reached by all of them.
// What bounds it is latency: one wave per SIMD and a chain of dependent steps,
// about 21,000 cycles for a chain of 150 atoms, of which the loads at the start
// take 2,700, the wrenches and torques 5,200, the step 2,000, the angles and the
// transform scan 4,700, the placement 1,400, the grid 2,400 and the cell list
// 2,800.  8.8 us in place of 47 us for the eight kernels it replaces (43 us with
// them in one graph).  What it took before: 39,200 cycles with LDS permutes for
// every lane move; 36,200 where every barrier waited for the stores before it,
// every look at the descriptor was a load and one thread sized the grid (13.9
// us); 26,500 where every atom compared itself with all of its cell (10.9 us);
// 24,000 where the torques went through LDS to a thread for each joint (10.3
// us).  768-thread form, 256 chains of 500 to 6,000 atoms: 108 us, 123 before
// the barriers changed.  Workgroups of 768 threads at most: 1,024 leave 128
// registers, where the form that keeps its loads needs 155 (32 spilled).
// SMALL, the form of at most 256 atoms, has one block of atoms and all joints
// in one wave: the thread of a joint's first atom has its whole torque, the
// scan needs no carries and no barrier before it, and another wave writes the
// axes.
template <int NT, bool ONE>
__global__ __launch_bounds__(NT) void k_chain(Batch bt, int mode)
{
    static_assert(JOINT_BLOCK == ATOM_BLOCK && NT % ATOM_BLOCK == 0, "blocks of one size");
    constexpr int NW = NT / WAVE, WPB = ATOM_BLOCK / WAVE;  // waves, waves per block
    constexpr bool KEEP_AXIS = ONE && NT <= 512;            // registers left for ua_1, pa_1
    constexpr bool SMALL = NT == 256;
    extern __shared__ __align__(16) unsigned char s_dyn[];
    __shared__ double s_red[NW][12];
    __shared__ double s_blk[CHAIN_JBLOCKS][12], s_carry[CHAIN_JBLOCKS][12];
    __shared__ double s_tm[NW];
    __shared__ double s_tau1[SMALL ? 3 * (NT / APR) : 1];
    __shared__ int s_bad[NW], s_scan[NW];

    ChainDev *dev = bt.n_chains == 1 ? bt.only : bt.table[blockIdx.x];
    ChainStats *st = stats_of(dev);
    const ChainView view(dev), *cd = &view;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), w = tid / WAVE;
    const int grp = tid / ATOM_BLOCK, gt = tid & (ATOM_BLOCK - 1), w0 = w & ~(WPB - 1);  // block in the pass, its first wave
    const bool lead = tid == 0;
    const int n = cd->n_atoms, J = cd->n_joints, n_chi = cd->n_chi;
    const int nblk = (n + ATOM_BLOCK - 1) / ATOM_BLOCK, njb = cd->n_bb_blocks;
    // flags and limits, read by every thread before any of them is written
    const bool active = st->active, pending = active && st->pending_post, fresh = st->need_grid;
    const bool grid_bad = st->grid_bad;
    const double tol = st->tol;
    const int64_t it1 = st->iterations + 1, it_limit = st->iter_limit;
    const int overflow = st->nbr_overflow;
    int go = st->run;
    asm volatile("" : : "v"(go), "v"(overflow), "v"(tol), "v"(it1), "v"(it_limit), "v"((int)grid_bad), "v"((int)fresh));
    // a thread with one atom and one joint takes what it needs of them now, all
    // loads in flight together, and keeps it
    // (threads beyond the last atom or joint the last one's, and leave it)
    double4 r0_1, ap_1, u0_1, p0_1, uc_1, pc_1, ua_1, pa_1;  // ua, pa: axis of the joint whose first atom this is
    double th_1 = 0.0;
    unsigned free_1 = 0, free_a = 0;  // whether joint tid moves; the joint of atom tid
    AtomForce in_1;  // stale, and not used, unless pending
    if (ONE) {
        // (SMALL: each wave has all joints)
        const int a = min(tid, n - 1), j = min(SMALL ? lane : tid, J - 1), res = a / APR, slot = a - res * APR;
        const int ja = 2 * res + (slot == 8 ? 1 : 0);
        in_1 = load_force(cd, a);
        if (KEEP_AXIS) {
            ua_1 = cd->jcur[2 * ja];
            pa_1 = cd->jcur[2 * ja + 1];
        }
        if (SMALL) {
            free_a = cd->mask[slot == 4 && n_chi ? J + res : ja];
        } else {
            uc_1 = cd->jcur[2 * j];
            pc_1 = cd->jcur[2 * j + 1];
        }
        u0_1 = cd->joint0[2 * j];
        p0_1 = cd->joint0[2 * j + 1];
        th_1 = cd->theta[min(tid, J + n_chi - 1)];
        free_1 = cd->mask[min(tid, J + n_chi - 1)];
        r0_1 = cd->r0[a];
        ap_1 = cd->aparam[a];
    }
    const GridRule rule = grid_rule(cd);
    unsigned *s_cell = reinterpret_cast<unsigned *>(s_dyn + (ONE ? sizeof(double) * 12 * (J + 1) : 0));
    if (ONE) {
        for (int i = tid; i < rule.cap_cells / (SMALL ? 4 : 8); i += NT) reinterpret_cast<uint4 *>(s_cell)[i] = make_uint4(0, 0, 0, 0);
        // here all the loads are done: a wait for one behind the stores below
        // would wait for those too
        auto done = [](double4 &v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z)); };
        done(u0_1); done(p0_1); done(r0_1); done(ap_1);
        if (!SMALL) { done(uc_1); done(pc_1); }
        if (KEEP_AXIS) { done(ua_1); done(pa_1); }
        asm volatile("" : "+v"(ap_1.w), "+v"(th_1), "+v"(free_1), "+v"(free_a));
    }
    // Before the first thread of the workgroup changes a flag a barrier follows
    // the reads above.  Barriers are of LDS only, as nothing else goes between
    // threads, but for the side-chain angles.
    if (mode == MODE_TAU && !pending) return;
    if (!active) {
        lds_barrier();
        if (lead) {
            st->pending_post = 0;
            if (mode == MODE_FINAL) st->active = running(st);
        }
        return;
    }

    double tm = 0.0;
    if (pending) {
        int bad = 0;
        double *s_tau = SMALL ? s_tau1 : reinterpret_cast<double *>(s_dyn);
        if (SMALL) {
            // one block of atoms: the thread of a joint's first atom has its whole torque
            double4 r;
            double S[WPART];
            wrench_of(in_1, tid < n, r, S);
            wave_suffix(S);
            if (lane == 0)
#pragma unroll
                for (int k = 0; k < WPART; ++k) s_red[w][k] = S[k];
            lds_barrier();
            add_later_waves<WPB>(S, s_red, w);
            const int res = tid / APR, slot = tid - res * APR;
            const bool axis = slot == 2 || slot == 8;
            if (tid < n && (axis || (slot == 4 && n_chi))) {
                const double t = axis ? axis_torque(ua_1, pa_1, S) + 0.0 : chi_torque(cd, tid, r);
                const int j = axis ? 2 * res + (slot == 8 ? 1 : 0) : J + res;
                s_tau[j] = t;
                cd->tau[j] = t;
                bad = !isfinite(t);
                if (free_a) tm = fabs(t);
            }
            tm = wave_max(tm);
            bad = __any(bad);
            if (w == NW - 1) {
                // (the last wave has the fewest atoms) energies and the
                // non-finite force flag of the pending forces, one to a lane
                double e = 0.0;
#pragma unroll
                for (int i = 0; i < NW; ++i) e += s_red[i][6 + (lane & 3)];
                if (lane == 0) st->e_elec = e;
                if (lane == 1) st->e_vdw = e;
                if (lane == 2) st->e_cav = e;
                if (lane == 3) st->post_bad = e > 0.0 ? 1 : 0;
                bad = bad || __any(lane == 3 && e > 0.0);
            }
            if (lane == 0) {
                s_tm[w] = tm;
                s_bad[w] = bad;
            }
            lds_barrier();
        } else {
            // wrenches and torques: s_tau[j] first holds the part of tau_j from the
            // atom block of j's first downstream atom, s_part the block sums
            double(*s_part)[WPART] = reinterpret_cast<double(*)[WPART]>(s_tau + J + n_chi);
            for (int lb0 = 0; lb0 < nblk; lb0 += NT / ATOM_BLOCK) {
                const int lb = lb0 + grp, a = lb * ATOM_BLOCK + gt;
                double4 r;
                double S[WPART];
                wrench_of(ONE ? in_1 : load_force(cd, min(a, n - 1)), a < n, r, S);
                wave_suffix(S);
                if (!ONE) lds_barrier();  // the last pass has read s_red
                if (lane == 0)
#pragma unroll
                    for (int k = 0; k < WPART; ++k) s_red[w][k] = S[k];
                lds_barrier();
                add_later_waves<WPB>(S, s_red + w0, w - w0);
                if (a < n) {
                    const int res = a / APR, slot = a - res * APR;
                    if (slot == 4 && n_chi) s_tau[J + res] = chi_torque(cd, a, r);
                    if (slot == 2 || slot == 8) {
                        const int j = 2 * res + (slot == 8 ? 1 : 0);
                        s_tau[j] = KEEP_AXIS ? axis_torque(ua_1, pa_1, S) : joint_torque(cd, j, S);
                    }
                }
                if (gt < WPART && lb < nblk) {
                    double t = 0.0;
#pragma unroll
                    for (int i = 0; i < WPB; ++i) t += s_red[w0 + i][gt];
                    s_part[lb][gt] = t;
                }
            }
            lds_barrier();
            for (int j0 = 0; j0 < J; j0 += NT) {
                const int j = j0 + tid, jlo = j - gt;
                if (jlo + (w - w0) * WAVE < J) {  // the wave holds a joint
                    const int jhi = min(J, jlo + JOINT_BLOCK) - 1, bhi = first_atom_of_joint(jhi) / ATOM_BLOCK;
                    // wrench of the atom blocks after bhi, then of those down to j's
                    double S[6] = {0, 0, 0, 0, 0, 0};
                    if (bhi + 1 < nblk) {
                        static_assert(CHAIN_ATOMS <= ATOM_BLOCK * WAVE, "later blocks fit one wave");
                        const int b = bhi + 1 + lane;
#pragma unroll
                        for (int k = 0; k < 6; ++k) S[k] = wave_sum(b < nblk ? s_part[b][k] : 0.0);
                    }
                    if (j < J) {
                        for (int b = bhi; b > first_atom_of_joint(j) / ATOM_BLOCK; --b)
#pragma unroll
                            for (int k = 0; k < 6; ++k) S[k] += s_part[b][k];
                        const double t = s_tau[j] + (ONE ? axis_torque(uc_1, pc_1, S) : joint_torque(cd, j, S));
                        s_tau[j] = t;
                        cd->tau[j] = t;
                        if (!isfinite(t)) bad = 1;
                        if (ONE ? free_1 : cd->mask[j]) tm = fmax(tm, fabs(t));
                    }
                }
            }
            for (int j = tid; j < J + n_chi; j += NT) {
                if (j < J) continue;
                const double t = s_tau[j];
                cd->tau[j] = t;
                if (!isfinite(t)) bad = 1;
                if (ONE ? free_1 : cd->mask[j]) tm = fmax(tm, fabs(t));
            }
            tm = wave_max(tm);
            if (lane == 0) s_tm[w] = tm;
            bad = __any(bad);
            if (w == NW - 1) {
                // (the last wave has the fewest joints) energies and the non-finite force flag of the pending forces
                double E[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) E[k] = wave_sum(lane < nblk ? s_part[lane][6 + k] : 0.0);
                if (lane == 0) {
                    st->e_elec = E[0];
                    st->e_vdw = E[1];
                    st->e_cav = E[2];
                    st->post_bad = E[3] > 0.0 ? 1 : 0;
                }
                bad = bad || E[3] > 0.0;
            }
            if (lane == 0) s_bad[w] = bad;
            lds_barrier();
        }
        if (mode == MODE_TAU) return;
        bad = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) {
            tm = fmax(tm, s_tm[i]);
            bad |= s_bad[i];
        }
        if (bad) {
            if (lead) {
                st->status = -4;
                st->run = 0;
                st->pending_post = 0;
                st->active = 0;
            }
            return;
        }
        const double scale = step_scale(cd, tm), mxd = scale * tm;
        for (int j = tid; j < J + n_chi; j += NT) {
            const double d = (ONE ? free_1 : cd->mask[j]) ? scale * s_tau[j] : 0.0;
            cd->dtheta[j] = d;
            th_1 = stepped_angle(ONE ? th_1 : cd->theta[j], d);
            cd->theta[j] = th_1;
        }
        const bool conv = tol > 0.0 && mxd < tol;
        go = !conv && it1 < it_limit;
        if (lead) {
            st->max_tau = tm;
            st->max_dtheta = mxd;
            st->iterations = it1;
            if (overflow) st->status = -6;
            if (conv) st->converged = 1;
            st->run = go;
        }
    } else if (mode == MODE_ITER) {
        go = 1;
        lds_barrier();
        if (lead) st->run = 1;
    }
    const bool on = go && !grid_bad;
    if (mode == MODE_FINAL || !on) {
        if (lead) {
            st->pending_post = 0;
            st->active = on;
        }
        return;
    }
    // forward kinematics: s_G[j + 1] = T_jlo o ... o T_j inside each joint
    // block, then the products of the earlier blocks in front
    double(*s_G)[12] = reinterpret_cast<double(*)[12]>(s_dyn);
    if (SMALL) {
        static_assert(!SMALL || NT / APR * 2 <= WAVE, "one wave has all joints");
        if (w == 0) {
            Xf x = xf_identity();
            if (lane < J) x = joint_xf_of(u0_1, p0_1, th_1);
#pragma unroll
            for (int d = 1; d < WAVE; d <<= 1)
                if (d < J) {  // else there is nothing below to take
                    const Xf y = xf_from_below(x, d);
                    if (lane >= d) {
                        masked_branch();
                        x = xf_mul(y, x);
                    }
                }
            x = xf_mul(xf_identity(), x);  // no block in front (the product keeps its zeros' signs)
            if (lane < J) xf_store(s_G[lane + 1], x);
            if (lead) xf_store(s_G[0], xf_identity());
        }
        if (n_chi) __syncthreads();  // the side-chain angles are written
        else lds_barrier();
        if (w == NW - 1 && lane < J) fk_emit(xf_load(s_G[lane + 1]), lane, u0_1, p0_1, cd->jcur);
    } else {
        if (n_chi) __syncthreads();  // the side-chain angles are written
        else lds_barrier();          // s_tau is read
        for (int j0 = 0; j0 < J; j0 += NT) {
            const int j = j0 + tid, jb = j / JOINT_BLOCK;
            const bool holds = j - lane < J;  // the wave holds a joint
            Xf x = xf_identity();
            if (holds) {
                if (j < J) {
                    if (!ONE) {
                        u0_1 = cd->joint0[2 * j];
                        p0_1 = cd->joint0[2 * j + 1];
                        th_1 = cd->theta[j];
                    }
                    x = joint_xf_of(u0_1, p0_1, th_1);
                }
                const int held = J - (j - lane);  // joints in the wave
#pragma unroll
                for (int d = 1; d < WAVE; d <<= 1)
                    if (d < held) {  // else there is nothing below to take
                        const Xf y = xf_from_below(x, d);
                        if (lane >= d) {
                            masked_branch();
                            x = xf_mul(y, x);
                        }
                    }
                if (lane == WAVE - 1) xf_store(s_red[w], x);
            }
            lds_barrier();
            if (holds) {
                if (w > w0) {
                    Xf pre = xf_load(s_red[w0]);
                    for (int i = w0 + 1; i < w; ++i) pre = xf_mul(pre, xf_load(s_red[i]));
                    x = xf_mul(pre, x);
                }
                if (ONE) x = xf_mul(xf_identity(), x);  // no block in front (the product keeps its zeros' signs)
                if (j < J) {
                    xf_store(s_G[j + 1], x);
                    if (ONE) fk_emit(x, j, u0_1, p0_1, cd->jcur);
                }
                if (!ONE && j == min(J, (jb + 1) * JOINT_BLOCK) - 1) xf_store(s_blk[jb], x);
            }
            if (!ONE) lds_barrier();
        }
        if (lead) xf_store(s_G[0], xf_identity());
        lds_barrier();
        if (!ONE && w == 0) {
            if (lane == 0) xf_store(s_carry[0], xf_identity());
            if (njb > 1) {
                Xf x = lane < njb - 1 ? xf_load(s_blk[lane]) : xf_identity();
                static_assert(CHAIN_JBLOCKS <= 8, "carries of at most eight blocks");
#pragma unroll
                for (int d = 1; d < 8; d <<= 1) {
                    Xf y = xf_from_below(x, d);
                    if (lane >= d) {
                        masked_branch();
                        x = xf_mul(y, x);
                    }
                }
                if (lane < njb - 1) xf_store(s_carry[lane + 1], x);
            }
        }
        if (!ONE) {
            lds_barrier();
            for (int j = tid; j < J; j += NT) {
                const Xf G = xf_mul(xf_load(s_carry[j / JOINT_BLOCK]), xf_load(s_G[j + 1]));
                xf_store(s_G[j + 1], G);
                fk_emit(G, j, cd->joint0[2 * j], cd->joint0[2 * j + 1], cd->jcur);
            }
            lds_barrier();
        }
    }

    // positions and bounding box
    double lo[3] = {DBL_MAX, DBL_MAX, DBL_MAX}, hi[3] = {-DBL_MAX, -DBL_MAX, -DBL_MAX};
    bool fin = true;
    double4 r1 = make_double4(0, 0, 0, 0);
    for (int a = tid; a < n; a += NT) {
        const double4 r = placed_atom(cd, a, ONE ? r0_1 : cd->r0[a], s_G[link_of_atom(a)]);
        cd->r[a] = r;
        if (ONE) r1 = r;
        cd->f_cav[3 * a] = 0;
        cd->f_cav[3 * a + 1] = 0;
        cd->f_cav[3 * a + 2] = 0;
        fin = fin && isfinite(r.x) && isfinite(r.y) && isfinite(r.z);
        lo[0] = fmin(lo[0], r.x); lo[1] = fmin(lo[1], r.y); lo[2] = fmin(lo[2], r.z);
        hi[0] = fmax(hi[0], r.x); hi[1] = fmax(hi[1], r.y); hi[2] = fmax(hi[2], r.z);
    }
    wave_box(lo, hi);
    fin = !__any(!fin);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < 3; ++k) { s_red[w][k] = lo[k]; s_red[w][3 + k] = hi[k]; }
        s_bad[w] = fin ? 0 : 1;
    }
    lds_barrier();
    // every wave sizes the grid
    const int ax = min(lane, 2);
    double lo_a = DBL_MAX, hi_a = -DBL_MAX;
    bool ok = true;
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        lo_a = min_num(lo_a, s_red[i][ax]);
        hi_a = max_num(hi_a, s_red[i][3 + ax]);
        ok = ok && !s_bad[i];
    }
    const Grid g = size_grid(rule, lo_a, hi_a, ok);
    if (!ok) {
        // a conformation that never had a grid stops the chain before its
        // first iteration
        if (lead) {
            st->status = -4;
            if (fresh) st->run = 0;
            else st->grid_bad = 1;
            st->need_grid = 0;
            st->pending_post = 0;
            st->active = 0;
        }
        return;
    }
    if (tid == NT - WAVE) {
        *grid_of(dev) = g;
        st->need_grid = 0;
    }

    if (SMALL) {
        // Cell list of at most 256 atoms, one to a thread: the lanes of a wave
        // that share a cell by ballots over the bits of the key, one byte of
        // the cell's word for the count of each wave.  A slot is then the
        // cell's start, the counts of the waves before and the lanes of the
        // cell below this one, which is the stable order at once, without the
        // scatter and a look at every member of the cell (3,000 cycles less).
        const int nc = g.n_cells;
        unsigned short *s_start = reinterpret_cast<unsigned short *>(s_cell + cd->cap_cells);
        const bool valid = tid < n;
        const int key = valid ? cell_of(g, r1) : 0;
        unsigned long long same = ballot(valid);
        for (int bit = 1; bit < nc; bit <<= 1) {
            const unsigned long long ones = ballot(key & bit);
            same &= key & bit ? ones : ~ones;
        }
        const int rank = count_below(same);
        if (valid && rank == 0) reinterpret_cast<unsigned char *>(s_cell + key)[w] = (unsigned char)__popcll(same);
        lds_barrier();
        const int per = (nc + NT - 1) / NT, i0 = min(tid * per, nc), i1 = min(i0 + per, nc);
        int sum = 0;
#pragma unroll 4
        for (int i = i0; i < i1; ++i) sum = (int)__builtin_amdgcn_sad_u8(s_cell[i], 0u, (unsigned)sum);
        const int x = wave_scan_i(sum);
        if (lane == WAVE - 1) s_scan[w] = x;
        lds_barrier();
        int run = x - sum;
#pragma unroll
        for (int i = 0; i < NW; ++i) run += i < w ? s_scan[i] : 0;
#pragma unroll 4
        for (int i = i0; i < i1; ++i) {
            s_start[i] = (unsigned short)run;
            cd->cell_start[i] = run;
            run = (int)__builtin_amdgcn_sad_u8(s_cell[i], 0u, (unsigned)run);
        }
        if (lead) cd->cell_start[nc] = n;
        lds_barrier();
        if (valid) {
            const unsigned before = s_cell[key] & ((1u << (8 * w)) - 1u);
            const int pos = s_start[key] + (int)__builtin_amdgcn_sad_u8(before, 0u, (unsigned)rank);
            cd->s_idx[pos] = tid;
            cd->s_r[pos] = make_double4(r1.x, r1.y, r1.z, __longlong_as_double((long long)tid | ((long long)(tid / APR) << 32)));
            cd->s_p[pos] = sorted_param(cd, ap_1);
        }
    } else {
        // cell list: counts and starts two to a word
        const int nc = g.n_cells, nword = (nc + 1) / 2;
        unsigned short *s_ids = reinterpret_cast<unsigned short *>(s_cell + cd->cap_cells / 2);
        unsigned short *s_key = s_ids + n, *s_arr = s_key + n;  // unless each thread keeps its one atom's
        if (!ONE) {
            for (int i = tid; i < nword; i += NT) s_cell[i] = 0;
            lds_barrier();
        }
        int key1 = 0, arr1 = 0;
        for (int a = tid; a < n; a += NT) {
            const int key = cell_of(g, ONE ? r1 : cd->r[a]), sh = 16 * (key & 1);
            const int arr = (int)((atomicAdd(&s_cell[key >> 1], 1u << sh) >> sh) & 0xffffu);
            if (ONE) {
                key1 = key;
                arr1 = arr;
            } else {
                s_key[a] = (unsigned short)key;
                s_arr[a] = (unsigned short)arr;
            }
        }
        lds_barrier();
        {
            const int per = (nword + NT - 1) / NT, i0 = min(tid * per, nword), i1 = min(i0 + per, nword);
            int sum = 0;
            for (int i = i0; i < i1; ++i) sum += (int)(s_cell[i] & 0xffffu) + (int)(s_cell[i] >> 16);
            const int x = wave_scan_i(sum);
            if (lane == WAVE - 1) s_scan[w] = x;
            lds_barrier();
            int run = x - sum;
#pragma unroll
            for (int i = 0; i < NW; ++i) run += i < w ? s_scan[i] : 0;
            for (int i = i0; i < i1; ++i) {
                const unsigned v = s_cell[i];
                s_cell[i] = (unsigned)run | ((unsigned)(run + (int)(v & 0xffffu)) << 16);
                run += (int)(v & 0xffffu) + (int)(v >> 16);
            }
        }
        lds_barrier();
        auto start_of = [&](int c) -> int { return c < nc ? (int)((s_cell[c >> 1] >> (16 * (c & 1))) & 0xffffu) : n; };
        for (int c = tid; c <= nc; c += NT) cd->cell_start[c] = start_of(c);
        for (int a = tid; a < n; a += NT) s_ids[start_of(ONE ? key1 : s_key[a]) + (ONE ? arr1 : s_arr[a])] = (unsigned short)a;
        lds_barrier();
        for (int a = tid; a < n; a += NT) {
            // the stable slot: the members of the cell with a smaller index before it
            const int key = ONE ? key1 : s_key[a], b = start_of(key), e = start_of(key + 1);
            int pos = b;
            for (int s = b; s < e; s += 4)
#pragma unroll
                for (int k = 0; k < 4; ++k) pos += (s + k < e && s_ids[min(s + k, n - 1)] < a) ? 1 : 0;
            const double4 r = ONE ? r1 : cd->r[a];
            cd->s_idx[pos] = a;
            cd->s_r[pos] = make_double4(r.x, r.y, r.z, __longlong_as_double((long long)a | ((long long)(a / APR) << 32)));
            cd->s_p[pos] = sorted_param(cd, ONE ? ap_1 : cd->aparam[a]);
        }
    }
    if (lead) {
        // the force kernel follows: its forces await the next post phase
        st->active = 1;
        st->pending_post = 1;
    }
}

// The force kernel's view of a chain's descriptor: memory that no kernel writes,
// so that its pointers stay scalar loads also behind the kernel's stores and
// atomics, where a global load of the pointer would come first, and 64-bit
// address arithmetic with it.  256-chain batch 2,052 us, 2,116 without; 500
// short chains in water 197 and 208, FP64 275 and 291.
#if defined(__HIP_DEVICE_COMPILE__)
template <typename T> using cptr = const __attribute__((address_space(4))) T *;
#else
template <typename T> using cptr = const T *;
#endif
using CDev = cptr<ChainDev>;
// (So are the constants of an atom: read as scalars they need not wait for the
// atomics under way, as a vector load behind those does: 10,000 atoms 40.0 us,
// 41.2 so, the batch 2,009 and 2,038.)
template <typename T> __device__ __forceinline__ cptr<T> constant(const T *p) { return (cptr<T>)p; }
// fixed-point accumulation of the solvation force
__device__ __forceinline__ void fix_add(gptr<long long> p, long long v)
{
    __hip_atomic_fetch_add((gptr<unsigned long long>)p, (unsigned long long)v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// k_force: Coulomb + LJ + SASA enumeration, one wave per atom
// ---------------------------------------------------------------------------
// A solvation neighbour j of atom i: offset a = r_j - r_i and the threshold c0 =
// (R_i^2 + |a|^2 - R_j^2) / (2 R_i): sample q_k = r_i + R_i Q_k is covered by j iff
// Q_k . a >= c0 (the same test as ||q_k - r_j|| <= R_j).
template <typename Real>
struct NbrEntry {
    Real ax, ay, az, c0;
};

// One atom's parameters from s_p, at a byte offset.
template <typename Real>
struct AtomPar {
    Real q, R, se;
    double roff;
};
template <typename Real> __device__ __forceinline__ AtomPar<Real> load_par(gptr<const char> sp, unsigned ob);
template <> __device__ __forceinline__ AtomPar<float> load_par<float>(gptr<const char> sp, unsigned ob)
{
    const float4 f = *(const gptr<const float4>)(sp + ob);
    return {f.x, f.y, f.z, *(const gptr<const double>)(sp + ob + 24)};
}
template <> __device__ __forceinline__ AtomPar<double> load_par<double>(gptr<const char> sp, unsigned ob)
{
    const double4 p = *(const gptr<const double4>)(sp + ob);
    return {p.x, p.y, p.z, p.w};
}

// Squared distance and cap threshold of a candidate, with the fused steps
// written out: every path and launch shape that takes them rounds alike.
__device__ __forceinline__ double dist2(double dx, double dy, double dz)
{
#pragma clang fp contract(off)
    return fma(dz, dz, fma(dy, dy, dx * dx));
}
__device__ __forceinline__ double cap_c0(double roff_i, double d2, double rj, double inv_2roff)
{
#pragma clang fp contract(off)
    return fma(-rj, rj, fma(roff_i, roff_i, d2)) * inv_2roff;
}

constexpr int SPL = SAMPLE_PASS / WAVE;             // samples per lane in one pass
// Neighbours whose cap on the offset sphere is large (cosine of its angular
// radius, c0/|a|, below CAP_SPLIT) lead the list: step 1 then reaches two
// overlappers for every sample of a slot early and stops there.
constexpr float CAP_SPLIT = 0.6f;
// Launch shapes of the force kernel (kcm_set_force_variant): candidates each
// lane loads per trip of the candidate loop (CPT), the neighbours step 1
// reads as one block before it checks the slots' saturation (SATB), and the
// order of the atoms over the workgroups, which go to the 8 XCDs in turn: cell
// order; XCD-aware by chunks (each XCD takes chunks of XCD_CHUNK consecutive
// cell-ordered atoms in turn, so that its L2 serves a few regions of space and
// all XCDs see the same mix of atoms); or XCD-aware by eighths (XCD x takes the
// x-th contiguous eighth).  Force kernel in shapes 0 to 3, us: 256-chain batch
// 1,958, 1,972, 1,960, 2,012; 10,000-residue globule 260, 260, 259, 268; 500 short
// chains in water 175, 180, 175, 178; 256 in vacuum (FP64) 28.8, 30.4, 28.4,
// 28.8; sixteen chains, every fourth compact and the others extended or coils,
// 335, 340, 282, 342; four compact chains and then twelve extended ones 376,
// 376, 390, 386, in FP64 538, 534, 558, 547.  Eighths gain where dense and sparse
// chains alternate and lose where two XCDs get all of the dense ones; chunks are
// nowhere behind cell order by more than 1 %, and are the default.
// Every shape visits the candidates and appends the neighbours in the same
// order, and takes the same decisions: the results are the same bit for bit.
enum XcdOrder { CELL_ORDER, XCD_CHUNKS, XCD_EIGHTHS };
struct ForceShape {
    int cpt, satb;
    XcdOrder order;
};
constexpr ForceShape FORCE_SHAPES[] = {{1, 4, XCD_CHUNKS}, {1, 4, CELL_ORDER}, {1, 4, XCD_EIGHTHS}, {2, 4, XCD_CHUNKS}};
constexpr int XCD_CHUNK = 256;
constexpr int N_XCD = 8;
// Step-1 count of a sample: acc = (covering neighbours << ACC_SHIFT) + (sum of
// their slots), so acc >> ACC_SHIFT == 1 leaves the single overlapper in the
// low bits; slots below MAX_NBR keep the slot sum below 2^ACC_SHIFT.
constexpr int ACC_SHIFT = 17;
// After the first COMPACT_AT neighbours of the list, the samples of a pass
// that can still change (fewer than two overlappers so far, or a test inside
// the FP32 band) move to the leading slots, in sample order, and the others
// count as covered; the later blocks test only the slots that hold them.
// Each moves as one word in the unused end of the neighbour list: acc (below
// 2^STAGE_K: at most COMPACT_AT overlappers), its sample within the pass, and
// its band flag.
constexpr int COMPACT_AT = 16;
constexpr int STAGE_K = 22;
static_assert(COMPACT_AT * ((1 << ACC_SHIFT) + COMPACT_AT) < (1 << STAGE_K), "staged count field");
static_assert(WAVE * SPL <= 256 && STAGE_K + 8 < 31, "staged sample field");
static_assert(MAX_NBR * (MAX_NBR - 1) / 2 < (1 << ACC_SHIFT), "slot sum must stay below the count field");
static_assert(MAX_NBR * 2 < (1 << (31 - ACC_SHIFT)), "count field must not overflow");
static_assert((2 * MAX_REACH + 1) * (2 * MAX_REACH + 1) <= WAVE, "stencil rows must fit one wave");
// Net events of one neighbour and axis from one pass of at most 256 samples lie
// in [-256, 256]: the three axes share a word as ten-bit fields biased by 512
// (no carry or borrow leaves a field), scattered after each pass.  One word
// instead of two keeps the mixed form's LDS within five of the 1,280-byte
// granules it is allotted in (6,272 bytes with the pair queue), 24 waves to a CU:
// with 6,720 bytes it was six granules and 21 waves, the 256-chain batch 2,419 us against 2,289.
constexpr int EV_BITS = 10, EV_BIAS = 1 << (EV_BITS - 1), EV_MASK = (1 << EV_BITS) - 1;
constexpr unsigned EV_INIT = EV_BIAS | EV_BIAS << EV_BITS | EV_BIAS << (2 * EV_BITS);
static_assert(WAVE * SPL < EV_BIAS, "events of a pass fit their field");
__device__ __forceinline__ int ev_of(unsigned w, int axis) { return (int)(w >> (EV_BITS * axis) & EV_MASK) - EV_BIAS; }
__device__ __forceinline__ unsigned ev_word(int e0, int e1, int e2)
{
    return (unsigned)e0 + ((unsigned)e1 << EV_BITS) + ((unsigned)e2 << (2 * EV_BITS));
}

__device__ __forceinline__ float bcast(float x, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), l));
}
__device__ __forceinline__ double bcast(double x, int l)
{
    const long long b = __double_as_longlong(x);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(b & 0xffffffffll), l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// a * b + c for a, b below 2^24 (b wave-uniform) as one full-rate 24-bit
// multiply-add; the compiler otherwise may pick the quarter-rate 32-bit
// multiply when it cannot bound b.
__device__ __forceinline__ int mad_u24(int a, int b, int c)
{
    int r;
    asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(b), "v"(c));
    return r;
}

// Step-1 code of four tests t0..t3 of one sample against the neighbours of a
// block: the sum of 32 + q over the tests with t_q >= 0, from the words that
// hold their signs (of a double the upper one).  Two byte permutes gather the
// four sign bits as bytes (0xff for a negative test, selectors 9 and 11
// replicate the top bit of the low and the high source word), and a signed dot
// product with the bytes 32..35 subtracts 32 + q for each negative test from
// the sum over all four (134): three instructions, where compares and selects
// take twelve.  A test of exactly -0 counts as uncovered here.  In FP32 |t| = 0
// lies in the band, so its sample is decided again in FP64; in FP64 no test is
// -0, as the chain of fused steps starts from 0 - c0.
// FP64, 500 short chains in water: 290 us, 298 with compares and selects.
__device__ __forceinline__ int block_code(int t0, int t1, int t2, int t3)
{
    const unsigned lo = __builtin_amdgcn_perm((unsigned)t1, (unsigned)t0, 0x0c0c0b09u);
    const unsigned hi = __builtin_amdgcn_perm((unsigned)t3, (unsigned)t2, 0x0b090c0cu);
    constexpr int ALL = 4 * 32 + 0 + 1 + 2 + 3;
    return __builtin_amdgcn_sdot4((int)(lo | hi), 0x23222120, ALL, false);
}
__device__ __forceinline__ int sign_word(float t) { return __float_as_int(t); }
__device__ __forceinline__ int sign_word(double t) { return __double2hiint(t); }

// FP64 decision in absolute coordinates: is sample k of atom i covered by the
// offset sphere of atom aj, shifted by delta_r along axis s (s < 0: not
// shifted)?
__device__ __forceinline__ bool cover_exact(CDev cd, const double4 &ri, double roff_i, int k, int aj, int s)
{
    const double4 q = glob(cd->q64)[k];
    const double qx = ri.x + roff_i * q.x, qy = ri.y + roff_i * q.y, qz = ri.z + roff_i * q.z;
    double4 c = glob(cd->r)[aj];
    if (s == 0) c.x += cd->delta_r;
    if (s == 1) c.y += cd->delta_r;
    if (s == 2) c.z += cd->delta_r;
    const double rj = glob(cd->aparam)[aj].w;
    const double dx = qx - c.x, dy = qy - c.y, dz = qz - c.z;
    return dx * dx + dy * dy + dz * dz - rj * rj <= 0.0;
}

// Coverage by a displaced neighbour, v = (tested quantity) with threshold 0;
// the mixed form decides again in FP64 inside the band.
template <typename Real, bool MIXED>
__device__ __forceinline__ bool test_cover(Real v, CDev cd, const double4 &ri, double roff_i, int k, int aj, int s)
{
    bool hit = v >= (Real)0;
    if (MIXED) {
        if (fabsf((float)v) <= MIXED_BAND) hit = cover_exact(cd, ri, roff_i, k, aj, s);
    }
    return hit;
}

// The three displaced tests of one (sample, neighbour) pair are decided in
// the form's precision first; the mixed form then takes every test inside the
// band again in FP64, the three behind one branch.  band3: is any of them in
// the band.
__device__ __forceinline__ bool band3(float v0, float v1, float v2)
{
    return fminf(fabsf(v0), fminf(fabsf(v1), fabsf(v2))) <= MIXED_BAND;
}
template <typename Real>
__device__ __forceinline__ void load_q(CDev cd, int k, Real &x, Real &y, Real &z)
{
    if (sizeof(Real) == 4) {
        const float4 q = glob(cd->q32)[k];
        x = (Real)q.x; y = (Real)q.y; z = (Real)q.z;
    } else {
        const double4 q = glob(cd->q64)[k];
        x = (Real)q.x; y = (Real)q.y; z = (Real)q.z;
    }
}

// One lane's Coulomb + LJ sums over its candidates (the stencil rows of the
// calling wave), all in FP64.  Called, out of line, for an atom whose FP32
// pair terms left the FP32 range: atoms a few hundredths of an angstrom apart
// drive (D/d)^12 and the force past it.  Same candidates, cutoff decisions and
// weights as the force kernel (eqs 02, 03).
struct PairSums {
    double f[3];
    double e[2];
};
__device__ __noinline__ PairSums pair_terms_fp64(CDev cd, int si, int off, int rbase, int T, int nrows,
                                                 int res_i, uint32_t m12, uint32_t m13, uint32_t m14, int terms)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const double4 ri = glob(cd->s_r)[si];
    const double4 pa = glob(cd->aparam)[(int)__double_as_longlong(ri.w)];
    const double cut2 = cd->cutoff * cd->cutoff;
    const bool do_elec = terms & 1, do_vdw = terms & 2;
    PairSums out = {{0.0, 0.0, 0.0}, {0.0, 0.0}};
#pragma unroll 1
    for (int kb = 0; kb < T; kb += WAVE) {
        const int k = kb + lane;
        int lo = 0;
#pragma unroll
        for (int step = 32; step >= 1; step >>= 1) {
            const int t = lo + step;
            const int o = __shfl(off, t & (WAVE - 1), WAVE);
            if (t < nrows && o <= k) lo = t;
        }
        int sj = __shfl(rbase, lo, WAVE) + k;
        const bool ok = k < T && sj != si;
        if (k >= T) sj = si;
        const double4 rj = glob(cd->s_r)[sj];
        const double ddx = rj.x - ri.x, ddy = rj.y - ri.y, ddz = rj.z - ri.z;
        const double d2 = dist2(ddx, ddy, ddz);
        if (!(ok && d2 <= cut2)) continue;
        const double4 pj = glob(cd->aparam)[(int)__double_as_longlong(rj.w)];
        const long long wj = __double_as_longlong(rj.w);
        const int aj = (int)wj, res_j = (int)(wj >> 32), dres = res_j - res_i;
        double we = do_elec ? 1.0 : 0.0, wv = do_vdw ? 1.0 : 0.0;
        if (dres >= -1 && dres <= 1) {
            const uint32_t bit = 1u << ((dres + 1) * APR + (aj - res_j * APR));
            if (m12 & bit) { we = 0; wv = 0; }
            else if (m13 & bit) { we *= cd->w13; wv *= cd->w13; }
            else if (m14 & bit) { we *= cd->w14e; wv *= cd->w14v; }
        }
        if (we == 0.0 && wv == 0.0) continue;
        const double inv2 = 1.0 / d2;
        const double eel = we * cd->coulomb * pa.x * pj.x * inv2;
        const double D = pa.y + pj.y;
        const double s2 = D * D * inv2, s6 = s2 * s2 * s2, s12 = s6 * s6;
        const double eij = pa.z * pj.z;
        const double fsc = (2.0 * eel + 12.0 * wv * eij * (s12 - s6)) * inv2;
        out.f[0] -= fsc * ddx;
        out.f[1] -= fsc * ddy;
        out.f[2] -= fsc * ddz;
        out.e[0] += eel;
        out.e[1] += wv * eij * (s12 - 2.0 * s6);
    }
    return out;
}

// Solvation of one atom with more neighbours than the LDS list holds (dense
// self-overlaps of random starts).  Called, out of line, by the force kernel's
// wave for that atom; the common path keeps its list in LDS in one piece.
// The neighbours are numbered in candidate order, as the kernel numbers them,
// and taken in chunks of MAX_NBR, each enumerated again from the candidates
// (the wave's stencil rows: off, rbase, nrows, T) into the kernel's LDS
// arrays when needed.  Step 1 runs over every chunk; a sample's count
// saturates at 2 (only 0, 1 and more matter) and keeps the single
// overlapper's number.  Step 2 and the event scatter go chunk by chunk.  The
// decisions are those of one list, so the results are the same.
struct ChunkedSasa {
    int ncov;                 // covered samples of this lane
    int own[3];               // this lane's share of the atom's own net events per axis
};
struct ChunkArgs {
    int si, off, rbase, nrows, T, nn;
};
template <typename Real>
__device__ __noinline__ ChunkedSasa sasa_chunked(CDev cd, const ChunkArgs c, NbrEntry<Real> *s_nbr,
                                                 int *s_nbr_a, unsigned *s_ev)
{
    constexpr bool MIXED = sizeof(Real) == 4;
    const int lane = threadIdx.x & (WAVE - 1);
    // the atom's quantities, read again rather than passed (the call then
    // keeps few of the kernel's registers live)
    struct {
        int si, off, rbase, nrows, T, nn, N;
        double4 ri;
        double roff_i, inv_2roff, dr;
        long long qf;
    } a;
    a.si = c.si; a.off = c.off; a.rbase = c.rbase; a.nrows = c.nrows; a.T = c.T; a.nn = c.nn;
    a.N = cd->n_samples;
    a.ri = glob(cd->s_r)[c.si];
    a.roff_i = glob(cd->s_p)[c.si].w;
    a.inv_2roff = 0.5 / a.roff_i;
    a.dr = cd->delta_r;
    a.qf = glob(cd->qfix)[(int)__double_as_longlong(a.ri.w)];
    const Real drr = (Real)a.dr, kq = (Real)(a.dr * a.dr / (2.0 * a.roff_i)), k1 = (Real)(a.dr / a.roff_i);
    const Real guard = MIXED ? (Real)(2.0f * MIXED_BAND) : (Real)1e-9;
    ChunkedSasa out = {0, {0, 0, 0}};

    // neighbours numbered [lo, lo + len) into LDS positions 0 .. len-1
    auto enum_window = [&](int lo, int len) {
        int nb = 0;
#pragma unroll 1
        for (int kb = 0; kb < a.T; kb += WAVE) {
            const int k = kb + lane;
            int r = 0;
#pragma unroll
            for (int step = 32; step >= 1; step >>= 1) {
                const int t = r + step;
                const int o = __shfl(a.off, t & (WAVE - 1), WAVE);
                if (t < a.nrows && o <= k) r = t;
            }
            int sj = __shfl(a.rbase, r, WAVE) + k;
            const bool valid = k < a.T && sj != a.si;
            if (k >= a.T) sj = a.si;
            const double4 rj = glob(cd->s_r)[sj];
            const double4 pj = glob(cd->s_p)[sj];
            const double ddx = rj.x - a.ri.x, ddy = rj.y - a.ri.y, ddz = rj.z - a.ri.z;
            const double d2 = dist2(ddx, ddy, ddz);
            const double lim = a.roff_i + pj.w + a.dr;
            const bool in_cav = valid && d2 <= lim * lim;
            const unsigned long long m = ballot(in_cav);
            if (in_cav) {
                const int pos = nb + count_below(m) - lo;
                if (pos >= 0 && pos < len) {
                    NbrEntry<Real> e;
                    e.ax = (Real)ddx; e.ay = (Real)ddy; e.az = (Real)ddz;
                    e.c0 = (Real)cap_c0(a.roff_i, d2, pj.w, a.inv_2roff);
                    s_nbr[pos] = e;
                    s_nbr_a[pos] = (int)__double_as_longlong(rj.w);
                }
            }
            nb += __popcll(m);
        }
    };

#pragma unroll 1
    for (int kb = 0; kb < a.N; kb += WAVE * SPL) {
        Real Qx[SPL], Qy[SPL], Qz[SPL];
        int cnt[SPL], who[SPL];
#pragma unroll
        for (int i = 0; i < SPL; ++i) {
            const int k = kb + lane + WAVE * i;
            Qx[i] = Qy[i] = Qz[i] = (Real)0;
            if (k < a.N) load_q<Real>(cd, k, Qx[i], Qy[i], Qz[i]);
            cnt[i] = who[i] = 0;
        }
        // step 1 over every chunk
        for (int lo = 0; lo < a.nn; lo += MAX_NBR) {
            const int len = min(a.nn - lo, MAX_NBR);
            __syncthreads();
            enum_window(lo, len);
            __syncthreads();
            int acc[SPL];
            Real amin[SPL];
#pragma unroll
            for (int i = 0; i < SPL; ++i) {
                acc[i] = 0;
                amin[i] = (Real)1e30;
            }
            for (int u = 0; u < len; ++u) {
                const NbrEntry<Real> e = s_nbr[u];
                const int inc = (1 << ACC_SHIFT) + u;
#pragma unroll
                for (int i = 0; i < SPL; ++i) {
                    const Real t = fma(Qz[i], e.az, fma(Qy[i], e.ay, fma(Qx[i], e.ax, -e.c0)));
                    acc[i] += (t >= (Real)0) ? inc : 0;
                    if (MIXED) amin[i] = fmin(amin[i], fabs(t));
                }
            }
#pragma unroll
            for (int i = 0; i < SPL; ++i) {
                if (MIXED) {
                    // a test within the band of its threshold: the whole wave
                    // recounts that sample in FP64, one lane per neighbour
                    unsigned long long bm = ballot(kb + lane + WAVE * i < a.N && amin[i] <= (Real)MIXED_BAND);
                    while (bm) {
                        const int l = __ffsll((long long)bm) - 1;
                        bm &= bm - 1;
                        const int kl = kb + l + WAVE * i;
                        int part = 0;
                        for (int u = lane; u < len; u += WAVE)
                            if (cover_exact(cd, a.ri, a.roff_i, kl, s_nbr_a[u], -1)) part += (1 << ACC_SHIFT) + u;
                        part = wave_sum_i(part);
                        if (lane == l) acc[i] = part;
                    }
                }
                const int cc = acc[i] >> ACC_SHIFT;
                if (cc == 1) who[i] = lo + (acc[i] & ((1 << ACC_SHIFT) - 1));
                cnt[i] = min(cnt[i] + cc, 2);
            }
        }
#pragma unroll
        for (int i = 0; i < SPL; ++i)
            if (kb + lane + WAVE * i < a.N && cnt[i] >= 1) ++out.ncov;
        // step 2 and the events, chunk by chunk
        for (int lo = 0; lo < a.nn; lo += MAX_NBR) {
            const int len = min(a.nn - lo, MAX_NBR);
            __syncthreads();
            enum_window(lo, len);
            for (int u = lane; u < len; u += WAVE) {
                s_ev[u] = EV_INIT;
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < SPL; ++i) {
                const int k = kb + lane + WAVE * i;
                const bool valid = k < a.N;
                if (valid && cnt[i] == 1 && who[i] >= lo && who[i] < lo + len) {
                    // critically overlapped: only the overlapper's shifted copies can expose it
                    const int u = who[i] - lo;
                    const NbrEntry<Real> e = s_nbr[u];
                    const int aj = s_nbr_a[u];
                    const Real base = Qx[i] * e.ax + Qy[i] * e.ay + Qz[i] * e.az - e.c0 - kq;
                    const Real span = drr + k1 * fmax(fabs(e.ax), fmax(fabs(e.ay), fabs(e.az)));
                    if (base - span <= guard) {
                        const int n0 = !test_cover<Real, MIXED>(base + drr * Qx[i] - k1 * e.ax, cd, a.ri, a.roff_i, k, aj, 0);
                        const int n1 = !test_cover<Real, MIXED>(base + drr * Qy[i] - k1 * e.ay, cd, a.ri, a.roff_i, k, aj, 1);
                        const int n2 = !test_cover<Real, MIXED>(base + drr * Qz[i] - k1 * e.az, cd, a.ri, a.roff_i, k, aj, 2);
                        if (n0 | n1 | n2) atomicAdd(&s_ev[u], ev_word(n0, n1, n2));
                    }
                }
                // exposed samples: one lane per neighbour, the samples broadcast
                const unsigned long long em0 = ballot(valid && cnt[i] == 0);
                if (!em0) continue;
                for (int v = 0; WAVE * v < len; ++v) {
                    const int u = lane + WAVE * v;
                    const bool own = u < len;
                    const NbrEntry<Real> e = s_nbr[own ? u : 0];
                    const int aj = s_nbr_a[own ? u : 0];
                    const Real lim = -(drr + k1 * fmax(fabs(e.ax), fmax(fabs(e.ay), fabs(e.az)))) - guard;
                    int d0 = 0, d1 = 0, d2 = 0;
                    unsigned long long em = em0;
                    while (em) {
                        const int l = __ffsll((long long)em) - 1;
                        em &= em - 1;
                        const Real qx = bcast(Qx[i], l), qy = bcast(Qy[i], l), qz = bcast(Qz[i], l);
                        const Real base = qx * e.ax + qy * e.ay + qz * e.az - e.c0 - kq;
                        if (own && base >= lim) {
                            const int kx = kb + l + WAVE * i;
                            if (test_cover<Real, MIXED>(base + drr * qx - k1 * e.ax, cd, a.ri, a.roff_i, kx, aj, 0)) --d0;
                            if (test_cover<Real, MIXED>(base + drr * qy - k1 * e.ay, cd, a.ri, a.roff_i, kx, aj, 1)) --d1;
                            if (test_cover<Real, MIXED>(base + drr * qz - k1 * e.az, cd, a.ri, a.roff_i, kx, aj, 2)) --d2;
                        }
                    }
                    if (own && (d0 | d1 | d2)) atomicAdd(&s_ev[u], ev_word(d0, d1, d2));
                }
            }
            __syncthreads();
            // eq F_cav_patch: atom i gains G0_i ev / (N dr) per axis, neighbour j the opposite
            for (int u = lane; u < len; u += WAVE) {
                const unsigned w = s_ev[u];
                const int aj = s_nbr_a[u];
                const int ev[3] = {ev_of(w, 0), ev_of(w, 1), ev_of(w, 2)};
#pragma unroll
                for (int x = 0; x < 3; ++x) {
                    if (!ev[x]) continue;
                    out.own[x] += ev[x];
                    fix_add(&glob(cd->f_cav)[3 * aj + x], (-(long long)ev[x] * a.qf));
                }
            }
        }
    }
    return out;
}

// Mixed form: six waves per SIMD (80 registers, 6,272 bytes of LDS), which
// hides the latency of the candidate loads and LDS reads better than four
// waves with room to spare (3.06 against 3.39 ms on the 256-chain batch when
// measured, with a longer list); a seventh finds no LDS, which holds 25 waves
// of a CU.  The FP64 form: four (127 registers; its 10,112 bytes allow 16 waves
// per CU).  CAV false: no
// chain of the batch has the solvation term.  Without its list and tests
// eight waves fit a SIMD in either form, and the candidates go by without the
// neighbour test (FP64, 256 chains of 100 to 200 atoms: 27.4 us, 39.0 with the
// general kernel; the results are the same bit for bit).
constexpr int force_waves(bool fp32, bool cav) { return cav ? (fp32 ? 6 : 4) : 8; }
// LDS of a CU, and of one wave in the granules it is allotted in.
constexpr int CU_LDS = 160 * 1024, LDS_GRANULE = 1280;
constexpr int lds_granules(int bytes) { return (bytes + LDS_GRANULE - 1) / LDS_GRANULE * LDS_GRANULE; }
template <typename Real, int CPT, int SAT_CHECK, XcdOrder ORDER, bool CAV>
__global__ __launch_bounds__(WAVE, force_waves(sizeof(Real) == 4, CAV)) void k_force(Batch bt)
{
    static_assert(SAT_CHECK * (SAT_CHECK - 1) / 2 < 32 && 32 + SAT_CHECK <= 64, "block code of step 1");
    constexpr bool MIXED = sizeof(Real) == 4;
    constexpr int LIST = CAV ? MAX_NBR : 1;  // entries of the neighbour list
    __shared__ NbrEntry<Real> s_nbr[LIST];
    __shared__ int s_nbr_a[LIST];
    __shared__ __align__(16) unsigned s_word[CAV ? MAX_NBR + 2 * WAVE : WAVE + 4 * (3 * APR + 1) * sizeof(Real) / 4];
    static_assert(4 * force_waves(MIXED, CAV) * lds_granules(sizeof(s_nbr) + sizeof(s_nbr_a) + sizeof(s_word)) <= CU_LDS,
                  "LDS for the waves that the registers allow");
    unsigned *const s_ev = s_word;              // net events of each neighbour in this pass
    unsigned *const s_pair = s_word + LIST;     // (sample, neighbour) pairs that await their displaced tests

    int atom = blockIdx.x;
    if (ORDER != CELL_ORDER) {
        const int x = blockIdx.x % N_XCD, k = blockIdx.x / N_XCD;
        if (ORDER == XCD_EIGHTHS) {
            const int nq = bt.total_atoms / N_XCD, nr = bt.total_atoms % N_XCD;
            atom = x * nq + min(x, nr) + k;
        } else if (atom < bt.total_atoms / (N_XCD * XCD_CHUNK) * (N_XCD * XCD_CHUNK)) {
            atom = (k / XCD_CHUNK * N_XCD + x) * XCD_CHUNK + k % XCD_CHUNK;  // the last part stays in cell order
        }
    }
    // the atom's chain: from the map of the batch, the chain of the first atom
    // of each group and a step per chain border in it (two dependent loads
    // where a binary search over 256 chains takes nine)
    const ChainDev *dev = bt.only;
    int si = atom;
    if (bt.n_chains > 1) {
        int c = 0;
        if (bt.atom_chain) {
            c = bt.atom_chain[atom >> bt.atom_chain_shift];
            while (bt.atom_off[c + 1] <= atom) ++c;
        } else {
            c = find_block_owner(bt.atom_off, bt.n_chains, atom);
        }
        dev = glob(bt.table)[c];
        si = atom - bt.atom_off[c];
    }
    const CDev cd = (CDev)dev;
    const int lane = threadIdx.x;

    // flags and grid lie at fixed places behind the descriptor, and their loads
    // are issued with those of its pointers: the empty asm uses all of them
    // before the first branch (the compiler otherwise moves each behind it,
    // one wait after the other)
    const gptr<const ChainStats> st = (gptr<const ChainStats>)((gptr<const char>)dev + STATS_OFFSET);
    const Grid g = *(gptr<const Grid>)((gptr<const char>)dev + GRID_OFFSET);
    int run = st->run;
    const int bad = st->grid_bad;
    const gptr<const char> sr = (gptr<const char>)glob(cd->s_r), sp = (gptr<const char>)glob(cd->s_p);
    asm("" : "+s"(run) : "s"(bad), "s"(sr), "s"(sp), "s"(si), "s"(g.origin[0]), "s"(g.origin[1]), "s"(g.origin[2]),
                 "s"(g.cell), "s"(g.inv_cell), "s"(g.reach_len), "s"(g.dims[0]), "s"(g.dims[1]), "s"(g.dims[2]), "s"(g.reach));
    if (!run || bad) return;
    const double4 ri = *(const gptr<const double4>)(sr + (unsigned)si * (unsigned)sizeof(double4));
    const AtomPar<Real> pi = load_par<Real>(sp, (unsigned)si * (unsigned)sizeof(double4));
    const int ai = (int)__double_as_longlong(ri.w);
    const int dxn = g.dims[0], dyn = g.dims[1], dzn = g.dims[2];
    // the atom's cell, by the expression that sorted it (no key decoding)
    const double ux = (ri.x - g.origin[0]) * g.inv_cell, fx0 = floor(ux);
    const int cx0 = (int)fx0;
    const int cx = min(max(cx0, 0), dxn - 1);
    const int cy = min(max((int)floor((ri.y - g.origin[1]) * g.inv_cell), 0), dyn - 1);
    const int cz = min(max((int)floor((ri.z - g.origin[2]) * g.inv_cell), 0), dzn - 1);
    const int R = g.reach, side = 2 * R + 1, nrows = side * side;
    // lane = row_z * side + row_y; side <= 8 and lane < 64 keep the FP32
    // quotient at least 1/16 away from an integer, far above its rounding
    const int row_z = (int)(((float)lane + 0.5f) * __builtin_amdgcn_rcpf((float)side));
    const int row_y = lane - row_z * side;

    // stencil rows, one per lane: for each (dy, dz) one contiguous run of
    // cells along x, i.e. one contiguous run of the cell-ordered atoms.  The
    // run keeps only the cells that can hold an atom within reach of atom i:
    // a row whose y-z slab is farther than the reach is empty, and the x run
    // covers [x_i - ext, x_i + ext] with ext^2 = reach^2 - (y-z distance)^2.
    // The pad on the reach absorbs rounding.
    int beg = 0, cnt = 0;
    {
        const int y = cy + row_y - R, z = cz + row_z - R;
        // distance to the slab: to its near edge, nothing in the atom's own row
        const double ey = g.origin[1] + (y + (row_y < R ? 1 : 0)) * g.cell, ez = g.origin[2] + (z + (row_z < R ? 1 : 0)) * g.cell;
        const double gy = row_y == R ? 0.0 : ey - ri.y, gz = row_z == R ? 0.0 : ez - ri.z;
        const double reach = g.reach_len + 1e-6, rest = reach * reach - gy * gy - gz * gz;
        const bool row = lane < nrows && (unsigned)y < (unsigned)dyn && (unsigned)z < (unsigned)dzn && rest >= 0.0;
        // the run's ends in cells from the atom's own, in FP32 unless one lies
        // so near a border that FP64 might put it on the other side
        const float f = (float)(ux - fx0), e = __builtin_amdgcn_sqrtf((float)rest) * (float)g.inv_cell;
        const float lo = f - e, hi = f + e;
        constexpr float NEAR = 1e-4f;
        const bool tie = fminf(fabsf(lo - rintf(lo)), fabsf(hi - rintf(hi))) < NEAR;
        int xa = cx0 + (int)floorf(lo), xb = cx0 + (int)floorf(hi);
        if (ballot(row && tie)) {
            const double ext = sqrt(rest);
            xa = (int)floor((ri.x - ext - g.origin[0]) * g.inv_cell);
            xb = (int)floor((ri.x + ext - g.origin[0]) * g.inv_cell);
        }
        const int xl = max(max(0, cx - R), min(xa, dxn - 1));
        const int xh = min(min(dxn - 1, cx + R), max(xb, 0));
        if (row && xl <= xh) {
            const int base = (z * dyn + y) * dxn;
            beg = glob(cd->cell_start)[base + xl];
            cnt = glob(cd->cell_start)[base + xh + 1] - beg;
        }
    }
    int off = wave_scan_i(cnt);
    const int T = __builtin_amdgcn_readlane(off, WAVE - 1);
    off -= cnt;                   // first candidate number of this row
    const int rbase = beg - off;  // candidate number k of row t is sorted atom rbase_t + k

    const int terms = cd->terms;
    const bool do_elec = terms & 1, do_vdw = terms & 2, do_cav = CAV && (terms & 4);
    const bool do_pair = do_elec || do_vdw;
    const double cut2 = cd->cutoff * cd->cutoff;
    const double roff_i = pi.roff;
    const double inv_2roff = 0.5 / roff_i;
    const double dr = cd->delta_r;
    const int res_i = ai / APR, slot_i = ai - res_i * APR;
    const Real coul = (Real)cd->coulomb;
    const Real qi = pi.q, Ri = pi.R, sei = pi.se;

    // Pair weights of each atom of residues res_i - 1 .. res_i + 1 relative to
    // atom i, and of any other atom in the last entry: (elec weight x coul x
    // q_i, vdw weight, 12 x vdw weight), from the bond classes (two bits per
    // atom: 0 none, 1 1-2, 2 1-3, 3 1-4).  They lie behind the start bits below
    // (the words are free until the candidates are done).  A class of weight zero adds zeros: its
    // atoms lie at the fixed distances of bonds and bond angles.
    const unsigned long long cls_word = cd->cls_word[slot_i];
    struct __align__(16) PairWeights {
        Real el, vdw, vdw12, pad;
    };
    PairWeights *s_wtab = reinterpret_cast<PairWeights *>(s_word + WAVE);
    static_assert(sizeof(unsigned) * WAVE + sizeof(PairWeights) * (3 * APR + 1) <= sizeof(s_word), "start bits and weights");
    if (lane <= 3 * APR) {
        const int cls = lane < 3 * APR ? (int)(cls_word >> (2 * lane)) & 3 : 0;
        const Real we = MIXED ? (Real)cd->wtab32[2 * cls] : (Real)cd->wtab64[2 * cls];
        const Real wv = MIXED ? (Real)cd->wtab32[2 * cls + 1] : (Real)cd->wtab64[2 * cls + 1];
        s_wtab[lane] = {we * coul * qi, wv, (Real)12 * wv, (Real)0};
    }
    __builtin_amdgcn_wave_barrier();

    // Sorted atom of candidate kw + lane, one window of 64 candidates at a
    // time, windows in increasing order.  The non-empty rows' bases move to the
    // leading lanes, and one bit per candidate says where a row starts, 32 to a
    // lane for MAP_SPAN candidates (the bits are set in the event array, free
    // until the candidates are done).  A window's two words then tell every lane
    // how many rows have started up to its candidate, and the last of them is
    // its row: 10 vector instructions a window and one LDS permute.
    constexpr int MAP_SPAN = 32 * WAVE;
    const unsigned long long full = ballot(cnt > 0);
    const int row_base = __builtin_amdgcn_ds_permute(4 * (cnt > 0 ? count_below(full) : WAVE - 1), rbase);
    unsigned starts = 0;  // this lane's word of start bits
    int started = 0;      // rows that start before the window
    auto window_atom = [&](int kw) -> int {
        const int w = (kw & (MAP_SPAN - 1)) >> 5;
        if (w == 0) {
            s_ev[lane] = 0;
            __builtin_amdgcn_wave_barrier();
            if (cnt > 0 && (unsigned)(off - kw) < (unsigned)MAP_SPAN) atomicOr(&s_ev[(off - kw) >> 5], 1u << (off & 31));
            __builtin_amdgcn_wave_barrier();
            starts = s_ev[lane];
        }
        const unsigned lo = __builtin_amdgcn_readlane(starts, w), hi = __builtin_amdgcn_readlane(starts, w + 1);
        // rows started at or below this lane: bit 0, then those at bits 1 .. lane
        const unsigned long long m = ((unsigned long long)hi << 32 | lo) >> 1;
        const int p = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, started + (int)(lo & 1) - 1));
        started += __popc(lo) + __popc(hi);
        return __builtin_amdgcn_ds_bpermute(4 * p, row_base) + kw + lane;
    };

    Real fx = 0, fy = 0, fz = 0;
    double ee = 0.0, evw = 0.0;
    int nn = 0, nfront = 0, nback = 0;
    // one candidate: pair terms into (fx, fy, fz, ee, evw); a solvation
    // neighbour with a large cap is appended at the front of the list, any
    // other at its back (growing down from MAX_NBR - 1), in lane order
    auto visit = [&](bool valid, const double4 &rj, const AtomPar<Real> &pj) {
        // contraction off, the fused steps written out: the loop bodies of
        // all launch shapes round alike
#pragma clang fp contract(off)
        const double ddx = rj.x - ri.x, ddy = rj.y - ri.y, ddz = rj.z - ri.z;
        const double d2 = dist2(ddx, ddy, ddz);
        const int aj = (int)__double_as_longlong(rj.w);
        if (valid && do_pair && d2 <= cut2) {
            // (dres + 1) APR + slot_j, in [0, 3 APR) iff |dres| <= 1
            const PairWeights wt = s_wtab[min((unsigned)(aj - APR * res_i + APR), 3u * APR)];
            const Real rx = (Real)ddx, ry = (Real)ddy, rz = (Real)ddz;
            // mixed form: hardware reciprocal (1 ulp), far inside the force tolerance
            const Real inv2 = MIXED ? (Real)__builtin_amdgcn_rcpf((float)d2) : (Real)1 / (Real)d2;
            // eq 02 with eps = k_d d: E = (C/k_d) q_i q_j / d^2
            const Real eel = wt.el * pj.q * inv2;
            // eq 03: E = eps_ij [(D/d)^12 - 2 (D/d)^6], D = R_i + R_j, eps_ij = sqrt(eps_i eps_j)
            const Real D = Ri + pj.R;
            const Real s2 = D * D * inv2, s6 = s2 * s2 * s2, s12 = s6 * s6;
            const Real eij = sei * pj.se;
            const Real elj = wt.vdw * eij * fma((Real)-2, s6, s12);
            // |F|/d along r_i - r_j: 2 E_elec/d^2 + 12 eps (s12 - s6)/d^2
            const Real fsc = fma((Real)2, eel, wt.vdw12 * eij * (s12 - s6)) * inv2;
            fx = fma(-fsc, rx, fx);
            fy = fma(-fsc, ry, fy);
            fz = fma(-fsc, rz, fz);
            ee += (double)eel;
            evw += (double)elj;
        }
        if (!CAV) return;
        bool in_cav = false, front = false;
        double c0 = 0.0;
        if (do_cav) {
            const double Rj = pj.roff;
            const double lim = roff_i + Rj + dr;
            in_cav = valid && d2 <= lim * lim;
            c0 = cap_c0(roff_i, d2, Rj, inv_2roff);
            // c0 < CAP_SPLIT |a|; FP32 will do, the list's order does not change results
            const float cf = (float)c0;
            front = cf * fabsf(cf) < (CAP_SPLIT * CAP_SPLIT) * (float)d2;
        }
        const unsigned long long mf = ballot(in_cav && front), mb = ballot(in_cav && !front);
        const int cf = __popcll(mf), cb = __popcll(mb);
        // past the list's capacity nothing more is written: the atom then
        // takes the chunked path, which enumerates its neighbours again
        if (in_cav && nfront + cf + nback + cb <= MAX_NBR) {
            const int pos = front ? nfront + count_below(mf) : MAX_NBR - 1 - nback - count_below(mb);
            NbrEntry<Real> e;
            e.ax = (Real)ddx; e.ay = (Real)ddy; e.az = (Real)ddz;
            e.c0 = (Real)c0;
            s_nbr[pos] = e;
            s_nbr_a[pos] = aj;
        }
        nfront += cf;
        nback += cb;
        nn += cf + cb;
    };

    // CPT candidates per lane per trip, every load issued before any is used.
    // Loads take 32-bit byte offsets from the chain's arrays (n < 2^26 atoms
    // of 32 bytes).
    // The sorted atoms of the next trip are found while this trip's loads are
    // in flight.
    int sj[CPT];
    auto map_trip = [&](int kb) {
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
            const int w = window_atom(kb + q * WAVE);  // wave-wide: every lane takes part
            sj[q] = kb + q * WAVE + lane < T ? w : si;
        }
    };
    if (T > 0) map_trip(0);
    for (int kb = 0; kb < T; kb += CPT * WAVE) {
        bool ok[CPT];
        double4 rj[CPT];
        AtomPar<Real> pj[CPT];
#pragma unroll
        for (int q = 0; q < CPT; ++q) {
            ok[q] = sj[q] != si;
            const unsigned ob = (unsigned)sj[q] * (unsigned)sizeof(double4);
            rj[q] = *(const gptr<const double4>)(sr + ob);
            pj[q] = load_par<Real>(sp, ob);
        }
        if (kb + CPT * WAVE < T) map_trip(kb + CPT * WAVE);
#pragma unroll
        for (int q = 0; q < CPT; ++q) visit(ok[q], rj[q], pj[q]);
    }

    // pair force and energies of atom i (each unordered pair is seen from both ends)
    double pv[5] = {(double)fx, (double)fy, (double)fz, ee, evw};
    const bool overflow = !(isfinite(pv[0]) && isfinite(pv[1]) && isfinite(pv[2]) && isfinite(ee) && isfinite(evw));
    if (MIXED && __any(overflow)) {
        // Atoms a few thousandths of an angstrom apart drive (D/d)^12 and the
        // force past the FP32 range: this atom's pair terms are taken again,
        // all in FP64 (a non-finite result then is a true one)
        const PairSums ps = pair_terms_fp64(cd, si, off, rbase, T, nrows, res_i, cd->m12[slot_i], cd->m13[slot_i],
                                            cd->m14[slot_i], terms);
        pv[0] = ps.f[0]; pv[1] = ps.f[1]; pv[2] = ps.f[2]; pv[3] = ps.e[0]; pv[4] = ps.e[1];
    }
    const double sums = wave_sum5(pv[0], pv[1], pv[2], pv[3], pv[4]);
    // stored now, so that nothing of the pair phase stays live below.  Both
    // pointers are read as scalars and the component comes from a table of four
    // bits for every eight lanes: the compiler otherwise makes one load at a
    // lane's own address of the two, and branches of the choices.
    const gptr<double> energies = (gptr<double>)glob(cd->e_atom) + 4 * (size_t)ai;
    if ((lane & 15) == 0 || lane == 8) {
        const gptr<double> forces = (gptr<double>)glob(cd->f_pair) + 4 * (size_t)ai;
        asm("" : : "s"(forces), "s"(energies));
        const int k = lane >> 3;
        const bool energy = 0x42 >> k & 1;  // lanes 8 and 48
        (energy ? energies : forces)[0x10210 >> 4 * k & 7] = energy ? 0.5 * sums : sums;
    }

    double e_cav = 0.0, n_exp = -1.0;
    if (do_cav) {
        // The overlapper's number must fit the low field of acc.
        if (nn >= (1 << ACC_SHIFT)) {
            if (lane == 0) cd->stats->nbr_overflow = 1;
            nn = 0;
        }
        const int nnc = min(nn, MAX_NBR);
        const int N = cd->n_samples;
        const Real drr = (Real)dr;
        // displaced copy of j along e_s covers the sample iff
        //   dot + dr Q_s - c0 - dr^2/(2 R_i) - (dr/R_i) a_s >= 0
        const Real kq = (Real)(dr * dr / (2.0 * roff_i)), k1 = (Real)(dr / roff_i);
        // The shift moves the tested value by drr Q_s - k1 a_s, at most
        // span = drr + k1 max_s |a_s| either way: an exposed sample whose
        // undisplaced value is below -span - guard stays exposed for every
        // axis, a critical one above span + guard stays covered, and their
        // three tests can be skipped with the same decisions.  guard holds
        // the FP32 decision band (mixed) or a rounding pad (FP64).
        const Real guard = MIXED ? (Real)(2.0f * MIXED_BAND) : (Real)1e-9;
        int ncov = 0;
        // net events of the atom itself per axis (the neighbours' reactions go
        // out at once); times the atom's quantum after the wave sum
        int own0 = 0, own1 = 0, own2 = 0;
        if (nn > MAX_NBR) {
            // more neighbours than the LDS list holds: chunks, out of line
            const ChunkArgs ca = {si, off, rbase, nrows, T, nn};
            const ChunkedSasa cs = sasa_chunked<Real>(cd, ca, s_nbr, s_nbr_a, s_ev);
            ncov = cs.ncov;
            own0 = cs.own[0];
            own1 = cs.own[1];
            own2 = cs.own[2];
        } else {
            // The list lies in two parts, large caps from 0 up and the others
            // from MAX_NBR - 1 down.  The front is filled up to a multiple of
            // SAT_CHECK from the lower end of the back, so that no block of
            // step 1 straddles the gap; neighbour u of the list then is entry
            // u below nf and u + gap from there on.
            const int nb_back = __builtin_amdgcn_readfirstlane(nback);
            int nf = __builtin_amdgcn_readfirstlane(nfront);
            {
                const int fill = min(-nf & (SAT_CHECK - 1), nb_back), src = MAX_NBR - nb_back + lane;
                if (lane < fill) {
                    // component by component, so that the entry stays in registers
                    const Real ex = s_nbr[src].ax, ey = s_nbr[src].ay, ez = s_nbr[src].az, ec = s_nbr[src].c0;
                    const int a = s_nbr_a[src];
                    s_nbr[nf + lane].ax = ex;
                    s_nbr[nf + lane].ay = ey;
                    s_nbr[nf + lane].az = ez;
                    s_nbr[nf + lane].c0 = ec;
                    s_nbr_a[nf + lane] = a;
                }
                nf += fill;
            }
            const int nlist = __builtin_amdgcn_readfirstlane(nnc), gap = MAX_NBR - nlist;
            auto entry_of = [&](int u) -> int { return u < nf ? u : u + gap; };
            for (int kb = 0; kb < N; kb += WAVE * SPL) {
                for (int u = lane; u < nlist; u += WAVE) s_ev[entry_of(u)] = EV_INIT;
                __syncthreads();
                // step 1: coverage counts of SPL samples per lane
                Real Qx[SPL], Qy[SPL], Qz[SPL], amin[SPL];
                int acc[SPL];
#pragma unroll
                for (int i = 0; i < SPL; ++i) {
                    // (the tables are padded to whole passes)
                    load_q<Real>(cd, kb + lane + WAVE * i, Qx[i], Qy[i], Qz[i]);
                    acc[i] = 0;
                    amin[i] = (Real)1e30;
                }
                // Blocks of SAT_CHECK neighbours, read once for the four slots.  Once
                // every sample of a slot has two overlappers (decisions
                // outside the FP32 band; a sample with a test inside it is
                // recounted below over the whole list) the rest of the list
                // cannot change its C, and the slot's tests stop; the block
                // loop stops when all four slots have.
                // bit i: slot i holds a sample that can still change (wave-uniform)
                int livem = 0;
#pragma unroll
                for (int i = 0; i < SPL; ++i) {
                    // a lane past N starts saturated, so that it never holds
                    // its slot back (its count is not used)
                    if (kb + lane + WAVE * i >= N) acc[i] = 2 << ACC_SHIFT;
                    if (kb + WAVE * i < N) livem |= 1 << i;
                }
                // one block of SAT_CHECK neighbours from u for the live slots
                auto block = [&](int ul) {
                    const int u = entry_of(ul);
                    NbrEntry<Real> e[SAT_CHECK];
#pragma unroll
                    for (int q = 0; q < SAT_CHECK; ++q) e[q] = s_nbr[u + q];
                    Real minus_c0[SAT_CHECK];
#pragma unroll
                    for (int q = 0; q < SAT_CHECK; ++q) minus_c0[q] = MIXED ? -e[q].c0 : (Real)0 - e[q].c0;
                    int next = 0;
                    const int lm = __builtin_amdgcn_readfirstlane(livem);
                    const int kmul = (1 << ACC_SHIFT) + u - 32;
#pragma unroll
                    for (int i = 0; i < SPL; ++i) {
                        if (!((lm >> i) & 1)) continue;
                        // blk: 32 per covering neighbour plus its index in
                        // the block; its count c = blk >> 5 then adds
                        // c ((1 << ACC_SHIFT) + u) + (blk - 32 c) to acc
                        Real t[SAT_CHECK];
#pragma unroll
                        for (int q = 0; q < SAT_CHECK; ++q) {
                            t[q] = fma(Qz[i], e[q].az, fma(Qy[i], e[q].ay, fma(Qx[i], e[q].ax, minus_c0[q])));
                            if (MIXED) amin[i] = fmin(amin[i], fabs(t[q]));
                        }
                        static_assert(SAT_CHECK == 4, "four sign bytes per word");
                        const int blk = block_code(sign_word(t[0]), sign_word(t[1]), sign_word(t[2]), sign_word(t[3]));
                        acc[i] = mad_u24(blk >> 5, kmul, acc[i] + blk);
                        if (ballot(acc[i] < (2 << ACC_SHIFT))) next |= 1 << i;
                    }
                    livem = next;
                };
                // kept < 0: slot i of lane l holds sample kb + l + WAVE i;
                // else the first `kept` staged samples fill the slots in order
                int kept = -1;
                const bool can_stage = gap * (int)sizeof(NbrEntry<Real>) >= WAVE * SPL * (int)sizeof(int);
                int *s_stage = reinterpret_cast<int *>(s_nbr + nf);
                int u = 0;
                for (; livem && u < COMPACT_AT && u + SAT_CHECK <= nlist; u += SAT_CHECK) block(u);
                if (livem && u == COMPACT_AT && u + SAT_CHECK <= nlist && can_stage) {
                    int pos = 0;
#pragma unroll
                    for (int i = 0; i < SPL; ++i) {
                        const int kl = lane + WAVE * i;
                        const bool valid = kb + kl < N;
                        const bool band = MIXED && amin[i] <= (Real)MIXED_BAND;
                        const bool keep = valid && (acc[i] < (2 << ACC_SHIFT) || band);
                        const unsigned long long m = ballot(keep);
                        if (keep) s_stage[pos + count_below(m)] = acc[i] | (kl << STAGE_K) | (band ? 1 << 30 : 0);
                        if (valid && !keep) ++ncov;
                        pos += __popcll(m);
                    }
                    kept = __builtin_amdgcn_readfirstlane(pos);
                    __builtin_amdgcn_wave_barrier();
                    int next = 0;
#pragma unroll
                    for (int i = 0; i < SPL; ++i) {
                        if (WAVE * i >= kept) break;  // nothing reads the slots past the staged samples
                        int p = lane + WAVE * i;
                        asm volatile("" : "+v"(p));  // recomputed here, not kept (and spilled) from the pass start
                        acc[i] = 2 << ACC_SHIFT;
                        amin[i] = (Real)1e30;
                        Qx[i] = Qy[i] = Qz[i] = (Real)0;
                        if (p < kept) {
                            const int w = s_stage[p];
                            acc[i] = w & ((1 << STAGE_K) - 1);
                            if (w >> 30) amin[i] = (Real)0;
                            load_q<Real>(cd, kb + ((w >> STAGE_K) & 255), Qx[i], Qy[i], Qz[i]);
                        }
                        if (ballot(acc[i] < (2 << ACC_SHIFT))) next |= 1 << i;
                    }
                    livem = __builtin_amdgcn_readfirstlane(next);
                }
                for (; livem && u + SAT_CHECK <= nlist; u += SAT_CHECK) block(u);
                if (!livem) u = nlist;
                const int lm = __builtin_amdgcn_readfirstlane(livem);
                for (; u < nlist; ++u) {
                    const int ue = entry_of(u);
                    const NbrEntry<Real> e = s_nbr[ue];
                    const int inc = (1 << ACC_SHIFT) + ue;
#pragma unroll
                    for (int i = 0; i < SPL; ++i) {
                        if (!((lm >> i) & 1)) continue;
                        const Real t = fma(Qz[i], e.az, fma(Qy[i], e.ay, fma(Qx[i], e.ax, -e.c0)));
                        acc[i] += (t >= (Real)0) ? inc : 0;
                        if (MIXED) amin[i] = fmin(amin[i], fabs(t));
                    }
                }
                // sample in slot place p (lane + WAVE slot)
                auto sample_at = [&](int p) -> int { return kb + (kept < 0 ? p : (s_stage[p] >> STAGE_K) & 255); };
                // Displaced tests, one (sample, neighbour) pair per lane: a
                // critically overlapped sample with its overlapper (the
                // events are the copies that no longer cover it), an exposed
                // one with a neighbour whose copies may reach it (the events
                // are those that do).  Pairs collect in a queue and are taken
                // when they fill the wave, and at the end of the pass.
                int nq = 0;
                auto take_pairs = [&](int n, int from) {
                    if (lane < n) {
                        const unsigned w = s_pair[from + lane];
                        const int u = w & 255, k = sample_at((w >> 8) & 255);
                        const bool crit = w >> 16;
                        const NbrEntry<Real> e = s_nbr[u];
                        Real qx, qy, qz;
                        load_q<Real>(cd, k, qx, qy, qz);
                        const Real base = fma(qz, e.az, fma(qy, e.ay, fma(qx, e.ax, -(e.c0 + kq))));
                        const Real v0 = fma(-k1, e.ax, fma(drr, qx, base));
                        const Real v1 = fma(-k1, e.ay, fma(drr, qy, base));
                        const Real v2 = fma(-k1, e.az, fma(drr, qz, base));
                        int h0 = v0 >= (Real)0, h1 = v1 >= (Real)0, h2 = v2 >= (Real)0;
                        if (MIXED && band3((float)v0, (float)v1, (float)v2)) {
                            const int aj = s_nbr_a[u];
                            if (fabsf((float)v0) <= MIXED_BAND) h0 = cover_exact(cd, ri, roff_i, k, aj, 0);
                            if (fabsf((float)v1) <= MIXED_BAND) h1 = cover_exact(cd, ri, roff_i, k, aj, 1);
                            if (fabsf((float)v2) <= MIXED_BAND) h2 = cover_exact(cd, ri, roff_i, k, aj, 2);
                        }
                        const unsigned ev = (crit ? ev_word(1, 1, 1) : 0u) - ev_word(h0, h1, h2);
                        if (ev) atomicAdd(&s_ev[u], ev);
                    }
                };
                auto push_pairs = [&](bool mine, unsigned long long m, unsigned word) {
                    if (mine) s_pair[nq + count_below(m)] = word;
                    nq += __popcll(m);
                    __builtin_amdgcn_wave_barrier();
                    if (nq >= WAVE) {
                        nq -= WAVE;
                        take_pairs(WAVE, nq);
                    }
                };
#pragma unroll
                for (int i = 0; i < SPL; ++i) {
                    const int held = kept < 0 ? N - kb : kept;  // places that hold a sample
                    if (WAVE * i >= held) break;
                    const bool valid = lane + WAVE * i < held;
                    if (MIXED) {
                        // a test within the band of its threshold: the whole wave
                        // recounts that sample in FP64, one lane per neighbour
                        unsigned long long bm = ballot(valid && amin[i] <= (Real)MIXED_BAND);
                        while (bm) {
                            const int l = __ffsll((long long)bm) - 1;
                            bm &= bm - 1;
                            const int kl = sample_at(l + WAVE * i);
                            int part = 0;
                            for (int u = lane; u < nlist; u += WAVE) {
                                const int ue = entry_of(u);
                                if (cover_exact(cd, ri, roff_i, kl, s_nbr_a[ue], -1)) part += (1 << ACC_SHIFT) + ue;
                            }
                            part = wave_sum_i(part);
                            if (lane == l) acc[i] = part;
                        }
                    }
                    const int C = acc[i] >> ACC_SHIFT;
                    if (valid && C >= 1) ++ncov;
                    int p = lane + WAVE * i;
                    asm volatile("" : "+v"(p));  // computed here, not kept from the pass start
                    const bool crit = valid && C == 1;
                    const unsigned long long cm = ballot(crit);
                    if (cm) push_pairs(crit, cm, (unsigned)(acc[i] & ((1 << ACC_SHIFT) - 1)) | (unsigned)p << 8 | 1u << 16);
                    // exposed samples: one lane per neighbour, the samples
                    // broadcast from their lanes
                    const unsigned long long em0 = ballot(valid && C == 0);
                    if (em0) {
#pragma unroll 1
                        for (int u0 = 0; u0 < nlist; u0 += WAVE) {
                            const bool own = u0 + lane < nlist;
                            const int u = own ? entry_of(u0 + lane) : 0;
                            const NbrEntry<Real> e = s_nbr[u];
                            // below lim no axis reaches the sample
                            const Real lim = own ? -(drr + k1 * fmax(fabs(e.ax), fmax(fabs(e.ay), fabs(e.az)))) - guard : (Real)1e30;
                            const Real cb = -(e.c0 + kq);
                            unsigned long long em = em0;
                            while (em) {
                                const int l = __ffsll((long long)em) - 1;
                                em &= em - 1;
                                const Real qx = bcast(Qx[i], l), qy = bcast(Qy[i], l), qz = bcast(Qz[i], l);
                                const bool near = fma(qz, e.az, fma(qy, e.ay, fma(qx, e.ax, cb))) >= lim;
                                const unsigned long long m = ballot(near);
                                if (m) push_pairs(near, m, (unsigned)u | (unsigned)(l + WAVE * i) << 8);
                            }
                        }
                    }
                }
                take_pairs(nq, 0);
                __syncthreads();
                // eq F_cav_patch: atom i gains G0_i ev / (N dr) per axis, neighbour j the opposite
                const long long qf = constant(cd->qfix)[ai];
                for (int ul = lane; ul < nlist; ul += WAVE) {
                    const int u = entry_of(ul);
                    const unsigned w = s_ev[u];
                    if (w == EV_INIT) continue;
                    const int e0 = ev_of(w, 0), e1 = ev_of(w, 1), e2 = ev_of(w, 2), aj = s_nbr_a[u];
                    own0 += e0;
                    own1 += e1;
                    own2 += e2;
                    if (e0) fix_add(&glob(cd->f_cav)[3 * aj + 0], (-(long long)e0 * qf));
                    if (e1) fix_add(&glob(cd->f_cav)[3 * aj + 1], (-(long long)e1 * qf));
                    if (e2) fix_add(&glob(cd->f_cav)[3 * aj + 2], (-(long long)e2 * qf));
                }
                __syncthreads();
            }
        }
        __syncthreads();
        const int tot = wave_sum4_i(ncov, own0, own1, own2);
        if ((lane & 15) == 0 && lane && tot)
            fix_add(&glob(cd->f_cav)[3 * ai + (lane == 32 ? 0 : lane == 16 ? 1 : 2)], (long long)tot * constant(cd->qfix)[ai]);
        e_cav = constant(cd->g0)[ai] * (double)(N - tot) / (double)N;  // eq G_cav_patch (lane 0)
        n_exp = (double)(N - tot);
    }
    if (lane == 0) ((gptr<double2>)energies)[1] = make_double2(e_cav, n_exp);
}

// ---------------------------------------------------------------------------
// k_wrench: per-atom wrench (F, r x F) (eqs KCM_01, KCM_02), the suffix sum
// inside each workgroup and the workgroup-local joint torques; the chain
// kernel adds the contribution of later workgroups
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(ATOM_BLOCK) void k_wrench(Batch bt)
{
    const Owner own = owner_of(bt, bt.blk_chain, bt.blk_off, blockIdx.x);
    ChainStats *st = stats_of(own.cd);
    const ChainView view(own.cd), *cd = &view;
    const int lb = blockIdx.x - own.first;
    __shared__ double s_w[ATOM_BLOCK / WAVE][WPART];
    constexpr int NW = ATOM_BLOCK / WAVE;
    const int a = lb * ATOM_BLOCK + threadIdx.x, ac = min(a, cd->n_atoms - 1);
    const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
    const int res = a / APR, slot = a - res * APR, j = 2 * res + (slot == 8 ? 1 : 0), jc = min(j, cd->n_joints - 1);
    const AtomForce in = load_force(cd, ac);
    const double4 u = cd->jcur[2 * jc], p = cd->jcur[2 * jc + 1];
    loaded(in.f, in.r, in.e, in.c[0], in.c[1], in.c[2], u, p);
    const bool go = running(st);
    if (lb == 0 && threadIdx.x == 0) {
        // end of the iteration: the chain stays active iff it ran, and its
        // forces await the post phase
        st->active = go;
        if (go) st->pending_post = 1;
    }
    if (!go) return;
    double4 r;
    double S[WPART];
    wrench_of(in, a < cd->n_atoms, r, S);
    wave_suffix(S);
    if (lane == 0)
#pragma unroll
        for (int k = 0; k < WPART; ++k) s_w[w][k] = S[k];
    lds_barrier();
    add_later_waves<NW>(S, s_w, w);
    if (a < cd->n_atoms) {
        if (slot == 4 && cd->n_chi) cd->tau[cd->n_joints + res] = chi_torque(cd, a, r);
        if (slot == 2 || slot == 8) cd->tau[j] = axis_torque(u, p, S);
    }
    if (threadIdx.x < WPART) {
        double t = 0.0;
#pragma unroll
        for (int i = 0; i < NW; ++i) t += s_w[i][threadIdx.x];
        cd->wrench_part[WPART * lb + threadIdx.x] = t;
    }
}

// ---------------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------------
hipError_t launch_tau(const Batch &b, hipStream_t s)
{
    if (b.total_jblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tau, dim3(b.total_jblocks), dim3(JOINT_BLOCK), 0, s, b);
    return hipGetLastError();
}

template <int NT, bool ONE>
static hipError_t launch_chain_form(const Batch &b, int mode, hipStream_t s)
{
    // the link transforms and the cell list, which starts as zeros where each
    // has its place (ONE) and follows in the same place where not
    const int n = b.max_atoms, links = 2 * (n / APR) + 1;
    const size_t xf = sizeof(double) * 12 * links,
                 cells = sizeof(uint16_t) * (size_t)(NT == 256 ? 3 * cell_capacity(n) : cell_capacity(n) + (ONE ? 1 : 3) * n);
    const size_t lds = ONE ? xf + cells : std::max(xf, cells);
    if (lds > 65536) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_chain<NT, ONE>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, CHAIN_LDS);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_chain<NT, ONE>), dim3(b.n_chains), dim3(NT), lds, s, b, mode);
    return hipGetLastError();
}

hipError_t launch_chain(const Batch &b, int mode, hipStream_t s)
{
    if (b.n_chains <= 0) return hipSuccess;
    if (b.max_atoms <= 256) return launch_chain_form<256, true>(b, mode, s);
    if (b.max_atoms <= 512) return launch_chain_form<512, true>(b, mode, s);
    if (b.max_atoms <= 768) return launch_chain_form<768, true>(b, mode, s);
    return launch_chain_form<768, false>(b, mode, s);
}

hipError_t launch_stepfk(const Batch &b, int mode, hipStream_t s)
{
    if (b.total_jblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_stepfk, dim3(b.total_jblocks), dim3(JOINT_BLOCK), 0, s, b, mode);
    return hipGetLastError();
}

hipError_t launch_gridboot(const Batch &b, hipStream_t s)
{
    if (b.n_chains <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gridboot, dim3(b.n_chains), dim3(CHAIN_THREADS), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_finish(const Batch &b, hipStream_t s)
{
    if (b.n_chains <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_finish, dim3((b.n_chains + 255) / 256), dim3(256), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_stats_gather(const Batch &b, ChainStats *out, unsigned *flag, unsigned seq, hipStream_t s)
{
    if (b.n_chains <= 0) return hipSuccess;
    const int blocks = flag ? 1 : (b.n_chains + 63) / 64;
    hipLaunchKernelGGL(k_stats_gather, dim3(blocks), dim3(b.n_chains > 16 ? 1024 : 256), 0, s, b, out, flag, seq);
    return hipGetLastError();
}

hipError_t launch_box_read(const BoxRead &what, double *out, unsigned *flags, unsigned seq, int blocks, hipStream_t s)
{
    int64_t total = 0;
    for (int64_t n : what.n) total += n;
    // up to four waves, a value to a thread: each wave waits for its own stores
    // to reach the host (reads of some 2,000 values: four waves 3.9 us, one to
    // four by eight values to a thread 4.5, sixteen 6.0)
    const int threads = blocks > 1 ? 1024 : (int)std::min<int64_t>(256, (total + WAVE - 1) / WAVE * WAVE);
    hipLaunchKernelGGL(k_box_read, dim3(blocks), dim3(threads), 0, s, what, out, flags, seq);
    return hipGetLastError();
}

hipError_t launch_fold_control(const Batch &b, int mode, double tol, int64_t max_iter, hipStream_t s)
{
    if (b.n_chains <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_fold_control, dim3((b.n_chains + 255) / 256), dim3(256), 0, s, b, mode, tol, max_iter);
    return hipGetLastError();
}

hipError_t launch_mc_propose(const Batch &b, int mode, const double *delta, const int64_t *delta_off, int trial,
                             hipStream_t s)
{
    if (b.total_jblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mc_propose, dim3(b.total_jblocks), dim3(JOINT_BLOCK), 0, s, b, mode, delta, delta_off,
                       trial);
    return hipGetLastError();
}

hipError_t launch_mc_decide(const Batch &b, int mode, const double *u, int n_trials, int trial, double kT,
                            hipStream_t s)
{
    if (b.n_chains <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mc_decide, dim3((b.n_chains + 255) / 256), dim3(256), 0, s, b, mode, u, n_trials, trial,
                       kT);
    return hipGetLastError();
}

hipError_t launch_mc_apply(const Batch &b, hipStream_t s)
{
    if (b.total_jblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_mc_apply, dim3(b.total_jblocks), dim3(JOINT_BLOCK), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_set_theta(const Batch &b, const double *theta, const int64_t *theta_off, hipStream_t s)
{
    if (b.total_jblocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_set_theta, dim3(b.total_jblocks), dim3(JOINT_BLOCK), 0, s, b, theta, theta_off);
    return hipGetLastError();
}

hipError_t launch_place(const Batch &b, int mode, hipStream_t s)
{
    if (b.total_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_place, dim3(b.total_blocks), dim3(ATOM_BLOCK), 0, s, b, mode);
    return hipGetLastError();
}

// Key workgroups (atoms / 256) from which the grid gets a launch of its own:
// the 256-chain batch (3,196) runs faster split, the 1000-residue globule (40)
// with the grid sized in every key workgroup.
constexpr int CELLKEY_SPLIT_BLOCKS = 512;

hipError_t launch_cellkey(const Batch &b, hipStream_t s)
{
    if (b.total_blocks <= 0) return hipSuccess;
    // the separate sizing launch pays off once the key workgroups are many
    if (b.total_blocks >= CELLKEY_SPLIT_BLOCKS) {
        hipLaunchKernelGGL(k_grid, dim3(b.n_chains), dim3(WAVE), 0, s, b);
        hipLaunchKernelGGL(k_cellkey<false>, dim3(b.total_blocks), dim3(ATOM_BLOCK), 0, s, b);
    } else {
        hipLaunchKernelGGL(k_cellkey<true>, dim3(b.total_blocks), dim3(ATOM_BLOCK), 0, s, b);
    }
    return hipGetLastError();
}

hipError_t launch_cellscan(const Batch &b, hipStream_t s)
{
    if (b.n_chains <= 0) return hipSuccess;
    if (b.total_scan_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_cellscan, dim3(b.total_scan_blocks), dim3(CHAIN_THREADS), 0, s, b);
    return hipGetLastError();
}

hipError_t launch_scatter(const Batch &b, hipStream_t s)
{
    if (b.total_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_scatter, dim3(b.total_blocks), dim3(ATOM_BLOCK), sizeof(int) * (b.max_scan_chunks + 1), s, b);
    return hipGetLastError();
}

hipError_t launch_rank(const Batch &b, hipStream_t s)
{
    if (b.total_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_rank, dim3(b.total_blocks), dim3(ATOM_BLOCK), sizeof(int) * (b.max_scan_chunks + 1), s, b);
    return hipGetLastError();
}

hipError_t launch_wrench(const Batch &b, hipStream_t s)
{
    if (b.total_blocks <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_wrench, dim3(b.total_blocks), dim3(ATOM_BLOCK), 0, s, b);
    return hipGetLastError();
}

template <int V, bool CAV>
void launch_force_shape(const Batch &b, int precision, hipStream_t s)
{
    constexpr int C = FORCE_SHAPES[V].cpt, S = FORCE_SHAPES[V].satb;
    constexpr XcdOrder X = FORCE_SHAPES[V].order;
    if (precision == 1)
        hipLaunchKernelGGL((k_force<float, C, S, X, CAV>), dim3(b.total_atoms), dim3(WAVE), 0, s, b);
    else
        hipLaunchKernelGGL((k_force<double, C, S, X, CAV>), dim3(b.total_atoms), dim3(WAVE), 0, s, b);
}
template <int V>
void launch_force_shape(const Batch &b, int precision, hipStream_t s)
{
    if (b.terms & 4) launch_force_shape<V, true>(b, precision, s);
    else launch_force_shape<V, false>(b, precision, s);
}

hipError_t launch_force(const Batch &b, int precision, int shape, hipStream_t s)
{
    if (b.total_atoms <= 0) return hipSuccess;
    static_assert(sizeof(FORCE_SHAPES) / sizeof(FORCE_SHAPES[0]) == FORCE_SHAPE_COUNT, "shape table");
    switch (shape) {
    case 1: launch_force_shape<1>(b, precision, s); break;
    case 2: launch_force_shape<2>(b, precision, s); break;
    case 3: launch_force_shape<3>(b, precision, s); break;
    default: launch_force_shape<0>(b, precision, s); break;
    }
    return hipGetLastError();
}

}  // namespace kcm

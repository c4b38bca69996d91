// gfx950 kernels of the displaced-probing hot path (arXiv:2106.01275):
// probe generation (eqs. (3)-(4)), the gauge-covariant stencil A p, the CG
// vector updates with FP64 reductions, FP64 reliable updates, the displaced
// contraction z^H P x (Sec. 3) and the adjoint force.
//
// Data layout.  A block of W right-hand sides (W a power of two) is stored
// site-major with the right-hand side innermost: element (site, colour a,
// lane j) at ((site * nc + a) * W + j), complex.  A workgroup of 256 threads
// covers a tile of 256 / W sites; thread (site, j) = (tid / W, tid % W).  The
// W lanes of a site read consecutive addresses (coalesced) and share the
// site's links, which are staged once per tile in LDS (W >= 16) and reused by
// all W right-hand sides.  Consecutive tiles form one contiguous chunk per
// workgroup, and chunks are assigned so that each XCD owns a contiguous part
// of the lattice (its L2 then serves the x1/x2/x3 neighbour re-reads).
//
// Reductions (dot products per right-hand side) accumulate in FP64 across
// sites and workgroups; with FP32 or BF16 storage a thread first sums the
// few products of one site (its colours and hops) in FP32, or up to 24
// elements in the vector kernels, before adding them to its FP64 total.
// Every workgroup writes its partial sums, and a finishing kernel with one
// workgroup per right-hand side adds them in a fixed order (deterministic)
// and runs the CG scalar epilogue (alpha, beta, convergence flags) on the
// device, so the host only reads a control word now and then.  The kernel
// boundary makes the partials visible; no device-scope fence is used (on
// this multi-XCD part such a fence writes back the whole L2 of the XCD).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "dp_internal.h"

namespace dp {

// ============================================================ storage types

struct bf16x2 {
    uint32_t v;  // low half: real part, high half: imaginary part
};

typedef __bf16 bf16v2 __attribute__((ext_vector_type(2)));

// two FP32 values rounded to nearest even into one bf16x2 word (low = a)
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    bf16v2 v;
    v.x = (__bf16)a;
    v.y = (__bf16)b;
    return __builtin_bit_cast(uint32_t, v);
}

// c + a.lo * b.lo + a.hi * b.hi for bf16x2 words a, b (FP32 accumulation)
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16v2, a), __builtin_bit_cast(bf16v2, b), c, false);
}

// Global-memory pointers.  A pointer that the compiler cannot trace to a
// kernel argument (one read from a slot descriptor) is a generic one to it,
// and generic (flat) accesses also count against the LDS wait counter, so
// that every wait for an LDS read waits for them too.  The accessors below
// cast to the global address space at each access (every vector, link and
// index array of this library is in global memory).
template <typename T>
using gp = __attribute__((address_space(1))) T *;

// (the value moves as raw bits: copying a class type binds a generic
// reference, which brings the flat access back)
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

template <typename T>
__device__ __forceinline__ T ldg(const T *p) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8 || sizeof(T) == 16, "4, 8 or 16 bytes");
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, *(gp<const uint32_t>)p);
    else if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, *(gp<const uint64_t>)p);
    else return __builtin_bit_cast(T, *(gp<const u32x4>)p);
}

template <typename T>
__device__ __forceinline__ void stg(T *p, const T &v) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8 || sizeof(T) == 16, "4, 8 or 16 bytes");
    if constexpr (sizeof(T) == 4) *(gp<uint32_t>)p = __builtin_bit_cast(uint32_t, v);
    else if constexpr (sizeof(T) == 8) *(gp<uint64_t>)p = __builtin_bit_cast(uint64_t, v);
    else *(gp<u32x4>)p = __builtin_bit_cast(u32x4, v);
}

// The same past the caches' normal retention (see the vector update).
template <typename T>
__device__ __forceinline__ T ldg_nt(const T *p) {
    if constexpr (sizeof(T) == 4) return __builtin_bit_cast(T, __builtin_nontemporal_load((gp<const uint32_t>)p));
    else if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_nontemporal_load((gp<const uint64_t>)p));
    else return __builtin_bit_cast(T, __builtin_nontemporal_load((gp<const u32x4>)p));
}

template <typename T>
__device__ __forceinline__ void stg_nt(T *p, const T &v) {
    if constexpr (sizeof(T) == 4) __builtin_nontemporal_store(__builtin_bit_cast(uint32_t, v), (gp<uint32_t>)p);
    else if constexpr (sizeof(T) == 8) __builtin_nontemporal_store(__builtin_bit_cast(uint64_t, v), (gp<uint64_t>)p);
    else __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), (gp<u32x4>)p);
}

template <typename S>
struct St;

template <>
struct St<double2> {
    using R = double;
    template <bool NT = false>
    __device__ static __forceinline__ void ld(const double2 *__restrict__ a, size_t i, R &re, R &im) {
        double2 v = NT ? ldg_nt(a + i) : ldg(a + i);
        re = v.x;
        im = v.y;
    }
    template <bool NT = false>
    __device__ static __forceinline__ void st(double2 *__restrict__ a, size_t i, R re, R im) {
        NT ? stg_nt(a + i, make_double2(re, im)) : stg(a + i, make_double2(re, im));
    }
    __device__ static __forceinline__ void round(R &, R &) {}
};

template <>
struct St<float2> {
    using R = float;
    template <bool NT = false>
    __device__ static __forceinline__ void ld(const float2 *__restrict__ a, size_t i, R &re, R &im) {
        float2 v = NT ? ldg_nt(a + i) : ldg(a + i);
        re = v.x;
        im = v.y;
    }
    template <bool NT = false>
    __device__ static __forceinline__ void st(float2 *__restrict__ a, size_t i, R re, R im) {
        NT ? stg_nt(a + i, make_float2(re, im)) : stg(a + i, make_float2(re, im));
    }
    __device__ static __forceinline__ void round(R &, R &) {}
};

template <>
struct St<bf16x2> {
    using R = float;
    template <bool NT = false>
    __device__ static __forceinline__ void ld(const bf16x2 *__restrict__ a, size_t i, R &re, R &im) {
        uint32_t v = NT ? ldg_nt(a + i).v : ldg(a + i).v;
        re = __uint_as_float(v << 16);
        im = __uint_as_float(v & 0xffff0000u);
    }
    template <bool NT = false>
    __device__ static __forceinline__ void st(bf16x2 *__restrict__ a, size_t i, R re, R im) {
        bf16x2 o;
        o.v = pack_bf16(re, im);
        NT ? stg_nt(a + i, o) : stg(a + i, o);
    }
    // the value a store followed by a load would give
    __device__ static __forceinline__ void round(R &re, R &im) {
        const uint32_t v = pack_bf16(re, im);
        re = __uint_as_float(v << 16);
        im = __uint_as_float(v & 0xffff0000u);
    }
};

// ============================================================ helpers

// The workgroups working on one lattice: this workgroup's index b among
// them and their number nb.  A standalone launch uses (blockIdx, gridDim);
// in a multi-instance launch each slot owns a range of workgroups (starting
// at a multiple of 8, so b % 8 is still the XCD).
struct Blk {
    int b, nb;
};

__device__ __forceinline__ Blk own_blk() { return Blk{(int)blockIdx.x, (int)gridDim.x}; }

__device__ __forceinline__ int logical_block(const Blk &bk) {
    // Workgroups are dispatched round-robin over the 8 XCDs; renumber them so
    // that XCD x runs the contiguous range of logical blocks [x*n/8, (x+1)*n/8).
    const int n = bk.nb, b = bk.b;
    if (n % 8) return b;
    return (b % 8) * (n / 8) + b / 8;
}

__device__ __forceinline__ void tile_range(const Blk &bk, int ntiles, int &t0, int &t1) {
    const int lb = logical_block(bk), n = bk.nb;
    t0 = (int)(((long long)lb * ntiles) / n);
    t1 = (int)(((long long)(lb + 1) * ntiles) / n);
}

// Site traversal of the stencil kernels.  XCD x (workgroups with
// blockIdx % 8 == x) owns the x0-slices [x*D0/8, (x+1)*D0/8) when D0 is a
// multiple of 8 (otherwise one eighth of the site range); its workgroups
// walk the slab in steps, all together: step k covers consecutive work
// items, item w mapping to site (x0_lo + w % n0) * V3 + w / n0 (x0
// varies fastest).  The sites in flight then form a compact window whose
// neighbours (x0 ones included) are read at nearly the same time, so they
// hit in the XCD's L2.  (Taking the (x1, x2, x3) columns in blocks of a
// few x2-rows instead, so that the x1-neighbour planes of a window are
// those just read, cut the stencil's fetched bytes at 32^4 by a tenth but
// not its time, which is set by load latency rather than bytes.)
//
// In even-odd order a launch covers one half (half 0 or 1), whose index order
// is that of the lattice with D3 / 2 sites along x3: the same walk over
// N / 2 sites and V3 / 2 sites per slice, from site off = half * N / 2.
struct SiteWalk {
    int items;      // work items of this XCD
    int n0, x0_lo;  // x0-slices of the slab (n0 == 0: plain range)
    int base;       // first site (plain range)
    int V3;         // sites per x0-slice
    int off;        // first site of the half
    int first, stride;  // first tile of this workgroup and tile stride
    int n0s;            // log2 n0 if n0 is a power of two, else -1
};

__device__ __forceinline__ SiteWalk site_walk(const Launch &L, const Blk &bk, int half = 0) {
    const Lat &lat = L.lat;
    SiteWalk w;
    const int nb = bk.nb, b = bk.b, N = L.ns;
    w.V3 = (lat.D[1] * lat.D[2] * lat.D[3]) >> lat.eo;
    w.off = half * N;
    if (nb >= 8 && nb % 8 == 0) {
        const int x = b % 8;
        w.first = b / 8;
        w.stride = nb / 8;
        if (lat.D[0] % 8 == 0) {
            w.n0 = lat.D[0] / 8;
            w.x0_lo = x * w.n0;
            w.items = w.n0 * w.V3;
            w.base = 0;
        } else {
            w.n0 = 0;
            w.x0_lo = 0;
            w.base = (int)(((long long)x * N) / 8);
            w.items = (int)(((long long)(x + 1) * N) / 8) - w.base;
        }
    } else {
        w.first = b;
        w.stride = nb;
        w.n0 = 0;
        w.x0_lo = 0;
        w.base = 0;
        w.items = N;
    }
    w.n0s = w.n0 > 0 && (w.n0 & (w.n0 - 1)) == 0 ? __builtin_ctz(w.n0) : -1;
    return w;
}

// (a shift and a mask where n0 is a power of two: the walk is taken for
// every staged link element; 32^4, FP32, W = 32: 1.4% off the stencil)
__device__ __forceinline__ int walk_site(const SiteWalk &w, int item) {
    if (w.n0 == 0) return w.off + w.base + item;
    if (w.n0s >= 0) return w.off + (w.x0_lo + (item & (w.n0 - 1))) * w.V3 + (item >> w.n0s);
    return w.off + (w.x0_lo + item % w.n0) * w.V3 + item / w.n0;
}

// ABI index of internal site s, and internal site of ABI index x (see Lat).
// The extents of an even-odd order are even, so the parity of x0 + x1 + x2 is
// that of the three quotients of the row number.
__device__ __forceinline__ int row_parity(const Lat &L, int row) {
    const int r1 = row / L.D[2];
    return (row + r1 + r1 / L.D[1]) & 1;
}
__device__ __forceinline__ int lex_of(const Lat &L, int s) {
    if (!L.eo) return s;
    const int nh = L.N >> 1, par = s >= nh, x = 2 * (s - par * nh);
    return x + ((row_parity(L, x / L.D[3]) + par) & 1);
}
__device__ __forceinline__ int site_of(const Lat &L, int x) {
    if (!L.eo) return x;
    return ((row_parity(L, x / L.D[3]) + x) & 1) * (L.N >> 1) + (x >> 1);
}

// tiles of the whole lattice (L.ntiles: of the sites a launch iterates on)
__device__ __forceinline__ int full_tiles(const Launch &L) {
    const int spt = kBlock >> L.logW;
    return (L.lat.N + spt - 1) / spt;
}

__device__ __forceinline__ unsigned long long mix64(unsigned long long z) {
    // SplitMix64 output function (Steele, Lea, Flood, OOPSLA 2014)
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// noise value z0(s, site, b) as (re, im) in {-1, 0, 1}
__device__ __forceinline__ void noise_at(unsigned long long seedmix, unsigned long long ctr, int kind, double &re,
                                         double &im) {
    const unsigned long long h = mix64(seedmix ^ ctr);
    const int top = (int)(h >> 63), nxt = (int)((h >> 62) & 1ull);
    if (kind == DP_NOISE_REAL_Z2) {
        re = top ? -1.0 : 1.0;
        im = 0.0;
    } else if (kind == DP_NOISE_Z2_COMPLEX) {
        re = top ? -1.0 : 1.0;
        im = nxt ? -1.0 : 1.0;
    } else {
        const int q = (int)(h >> 62);
        re = q == 0 ? 1.0 : (q == 2 ? -1.0 : 0.0);
        im = q == 1 ? 1.0 : (q == 3 ? -1.0 : 0.0);
    }
}

__device__ __forceinline__ void noise(unsigned long long seedmix, long long s, int N, int site, int nc,
                                      int b, int kind, double &re, double &im) {
    noise_at(seedmix,
             ((unsigned long long)s * (unsigned long long)N + (unsigned long long)site) * (unsigned long long)nc +
                 (unsigned long long)b,
             kind, re, im);
}

__device__ __forceinline__ int shift0(const Lat &L, int site, int p) {
    // site + p e0 on the torus (p may be negative)
    const int stride0 = L.D[1] * L.D[2] * L.D[3];
    const int x0 = site / stride0;
    int y0 = (x0 + p) % L.D[0];
    if (y0 < 0) y0 += L.D[0];
    return site + (y0 - x0) * stride0;
}

// The sample s, colour c and dilution index a that lane-enumeration index J
// stands for (J = ((s - sample0) * ncolors + c) * n_dil + a); computed once
// per lane, outside the site loops (64-bit divisions).
struct ProbeLane {
    long long s;
    int c, a;
};

__device__ __forceinline__ ProbeLane probe_lane(const ProbeGen &g, int nc, long long J) {
    const int ndil = g.dilute ? nc : 1;
    ProbeLane pl;
    pl.s = g.sample0 + J / ((long long)g.ncolors * ndil);
    pl.c = (int)((J / ndil) % g.ncolors);
    pl.a = (int)(J % ndil);
    return pl;
}

// value of that lane's probe at (site of ABI index `site`, colour b); 0
// outside its support
__device__ __forceinline__ void probe_at(const ProbeGen &g, unsigned long long seedmix, const Lat &L, int nc,
                                         const ProbeLane &pl, int site, int b, double &re, double &im) {
    re = 0.0;
    im = 0.0;
    const int x = g.shift ? shift0(L, site, -g.shift) : site;
    if (g.colors[x] != pl.c) return;
    if (g.dilute && b != pl.a) return;
    noise(seedmix, pl.s, L.N, x, nc, b, g.noise, re, im);
}

// probe value of lane-enumeration index J at (site, colour b); 0 outside
__device__ __forceinline__ void probe_value(const ProbeGen &g, unsigned long long seedmix, const Lat &L,
                                            int nc, long long J, int site, int b, double &re, double &im) {
    probe_at(g, seedmix, L, nc, probe_lane(g, nc, J), site, b, re, im);
}

// ------------------------------------------------------------ reductions

// Writes this workgroup's sums of NV values per lane to
// dst[(lane * nblk + b) * NV + v] (all threads call it once).
// Lane j = tid % W: the threads of one lane inside a wavefront are summed by
// a butterfly over the thread-index bits above log2 W, then the wavefronts
// in order through LDS (sm: NV * kBlock doubles); a fixed order.
template <int NV>
__device__ void block_partials_to(const Blk &bk, const double (&val)[NV], int W, int logW, double *dst, int nblk,
                                  double *sm) {
    const int tid = threadIdx.x;
    double v_[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        v_[v] = val[v];
        for (int off = W; off < 64; off <<= 1) v_[v] += __shfl_xor(v_[v], off, 64);
    }
    // per wavefront, threads 0 .. min(W, 64) - 1 hold the sums of their lanes
    const int per_wave = W < 64 ? W : 64;
    const int lane_in_wave = tid & 63;
    if (lane_in_wave < per_wave) {
#pragma unroll
        for (int v = 0; v < NV; ++v) sm[v * kBlock + (tid >> 6) * per_wave + lane_in_wave] = v_[v];
    }
    __syncthreads();
    if (tid < W) {
        // lane tid's wavefront sums: W < 64: one per wavefront at
        // w * W + tid; W >= 64: the wavefronts w with w * 64 + (tid % 64) = tid
        // mod W, i.e. entries tid, tid + W, ... of the packed array
        const int nsum = W < 64 ? kBlock / 64 : kBlock / W;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            double s = 0.0;
            for (int k = 0; k < nsum; ++k) s += sm[v * kBlock + k * W + tid];
            stg(dst + ((size_t)tid * nblk + bk.b) * NV + v, s);
        }
    }
}

// the same into rd.part1
template <int NV>
__device__ void block_partials(const Blk &bk, const double (&val)[NV], int W, int logW, const Red &rd, double *sm) {
    block_partials_to<NV>(bk, val, W, logW, rd.part1, rd.nblk, sm);
}

// Total over the nblk partial sums of one lane, srcA = the lane's [nblk][NA]
// block (and srcB its [nblk][NB] one, both in one pass: the latencies of the
// two loads and of the two reductions overlap), in a fixed order (the same on
// every call): thread tid adds partials tid, tid + kBlock, ... (four loads in
// flight), then a butterfly in each wavefront and the wavefronts in order.
// All threads call it; the totals are valid in thread 0.  sm: (NA + NB) *
// kBlock / 64 doubles.
template <int NA, int NB>
__device__ __forceinline__ void lane_totals(const double *srcA, const double *srcB, int nblk, double (&totA)[NA],
                                            double (&totB)[NB > 0 ? NB : 1], double *sm) {
    constexpr int kWaves = kBlock / 64, NV = NA + NB;
    const int tid = threadIdx.x;
    auto at = [&](int b, int v) {
        return v < NA ? srcA[(size_t)b * NA + v] : srcB[(size_t)b * NB + (v - NA)];
    };
    double s[NV], s2[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) s[v] = s2[v] = 0.0;
    int b = tid;
    for (; b + 3 * kBlock < nblk; b += 4 * kBlock) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const double a0 = at(b, v), a1 = at(b + kBlock, v), a2 = at(b + 2 * kBlock, v), a3 = at(b + 3 * kBlock, v);
            s[v] += a0 + a1;
            s2[v] += a2 + a3;
        }
    }
    for (; b < nblk; b += kBlock) {
#pragma unroll
        for (int v = 0; v < NV; ++v) s[v] += at(b, v);
    }
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        double x = s[v] + s2[v];
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
        if ((tid & 63) == 0) sm[v * kWaves + tid / 64] = x;
    }
    __syncthreads();
#pragma unroll
    for (int v = 0; v < NV; ++v) {
        double t = 0.0;
        for (int w = 0; w < kWaves; ++w) t += sm[v * kWaves + w];
        if (v < NA)
            totA[v] = t;
        else
            totB[v - NA] = t;
    }
}

template <int NV>
__device__ __forceinline__ void lane_total(const double *src, int nblk, double (&tot)[NV], double *sm) {
    double none[1];
    lane_totals<NV, 0>(src, nullptr, nblk, tot, none, sm);
}

// The same total by one wavefront alone (any wavefront of the workgroup;
// no LDS, no barrier): thread t adds partials t, t + 64, ..., then a
// butterfly; the totals are valid in every thread of the wavefront.  For the
// slots of the multi-instance engine, whose lanes have a few dozen partials
// each.
template <int NV>
__device__ __forceinline__ void lane_total_wave(const double *src, int nblk, double (&tot)[NV]) {
    const int t = threadIdx.x & 63;
#pragma unroll
    for (int v = 0; v < NV; ++v) tot[v] = 0.0;
    for (int b = t; b < nblk; b += 64) {
#pragma unroll
        for (int v = 0; v < NV; ++v) tot[v] += src[(size_t)b * NV + v];
    }
#pragma unroll
    for (int v = 0; v < NV; ++v)
        for (int off = 32; off > 0; off >>= 1) tot[v] += __shfl_xor(tot[v], off, 64);
}

// Epilogues of the finishing kernels.  Those marked (part2, NV = 2) total
// the |r|^2 and Re q^H p partials of the last vector update, initialisation
// or reliable update; kEpiTj and kEpiStatsP1 total rd.part1.
enum Epi { kEpiInit, kEpiCheck, kEpiRU, kEpiStats, kEpiStatsP1, kEpiTj, kEpiInitEo };

// One workgroup per lane: total of the lane's partials (fixed order), then
// the scalar epilogue of that lane (thread 0; only this workgroup reads or
// writes lane j's state).
//   kEpiInit (part2)   |b|^2: the lane's CG state from scratch
//   kEpiCheck (part2)  |r|^2 of the latest residual into rr; FP64: lanes
//                      that meet tol stop (before a host check)
//   kEpiRU (part2)     the FP64 true residual of a reliable update
//   kEpiStats (part2), kEpiStatsP1 (part1)  a norm into true_rr only
//   kEpiTj (part1, NV = 2)  a complex dot product into tj
//   kEpiInitEo (part1, NV = 4, and part2)  even-odd order: |b|^2 of the whole
//                      lattice is in part2, |r|^2 of the reduced system's first
//                      residual in part1 (the |q|^2 entry); part2 then gets
//                      that |r|^2, as if an update had written r
template <int NV, int EPI>
__device__ __forceinline__ void k_finish_body(int lane, const Red &rd, const CgState &cs) {
    __shared__ double sm[NV * kBlock / 64];
    const int tid = threadIdx.x;
    if constexpr (EPI == kEpiInitEo) {
        __shared__ double sm6[6 * kBlock / 64], rr_all;
        double t4[4], t2[2];
        lane_totals<4, 2>(rd.part1 + (size_t)lane * rd.nblk * 4, rd.part2 + (size_t)lane * rd.nblk * 2, rd.nblk, t4, t2,
                          sm6);
        if (tid == 0) {
            const double bb = t2[0], rr = t4[2];
            rr_all = rr;
            cs.bb[lane] = bb;
            cs.rr[lane] = rr;
            cs.qp[lane] = 0.0;
            cs.rr_ref[lane] = rr;
            cs.true_rr[lane] = rr;
            cs.alpha[lane] = 0.0;
            cs.beta[lane] = 0.0;
            cs.iters[lane] = 0;
            cs.active[lane] = bb > 0.0;
            cs.flags[lane] = bb > 0.0 ? 0 : kFlagConverged;
            if (cs.live && lane == 0) *cs.live = 1;  // iterate until a control kernel counts the lanes
        }
        __syncthreads();  // (every partial has been read, too)
        for (int b = tid; b < rd.nblk; b += kBlock) {
            rd.part2[((size_t)lane * rd.nblk + b) * 2] = b == 0 ? rr_all : 0.0;
            rd.part2[((size_t)lane * rd.nblk + b) * 2 + 1] = 0.0;
        }
        return;
    }
    constexpr bool kPart2 = EPI == kEpiInit || EPI == kEpiCheck || EPI == kEpiRU || EPI == kEpiStats;
    static_assert(!kPart2 || NV == 2, "part2 holds two values per lane and workgroup");
    const double *src = (kPart2 ? rd.part2 : rd.part1) + (size_t)lane * rd.nblk * NV;
    const int j = lane;
    // the lane's state that the epilogue reads, loaded before the partials
    // so that the two loads' latencies overlap
    constexpr bool kState = EPI == kEpiCheck || EPI == kEpiRU;
    double st_ref = 0.0, st_bb = 0.0;
    int st_active = 0, st_flags = 0;
    if (kState && tid == 0) {
        st_ref = cs.rr_ref[j];
        st_bb = cs.bb[j];
        st_active = cs.active[j];
        st_flags = cs.flags[j];
    }
    double tot[NV];
    lane_total<NV>(src, rd.nblk, tot, sm);
    if (tid != 0) return;
    const double t = tot[0];
    if (EPI == kEpiInit) {
        cs.bb[j] = t;
        cs.rr[j] = t;
        cs.qp[j] = 0.0;
        cs.rr_ref[j] = t;
        cs.true_rr[j] = t;
        cs.alpha[j] = 0.0;
        cs.beta[j] = 0.0;
        cs.iters[j] = 0;
        cs.active[j] = t > 0.0;
        cs.flags[j] = t > 0.0 ? 0 : kFlagConverged;
        if (cs.live && j == 0) *cs.live = 1;  // iterate until a control kernel counts the lanes
    } else if (EPI == kEpiCheck) {
        cs.rr[j] = t;
        cs.qp[j] = tot[NV - 1];
        if (cs.exact && st_active && t <= cs.tol2 * st_bb) {
            cs.active[j] = 0;
            cs.flags[j] = st_flags | kFlagConverged;
        }
    } else if (EPI == kEpiRU) {
        // the residual is the true one from here on (the direction was
        // continued, kept or restarted by the kernel that wrote it)
        cs.true_rr[j] = t;
        if (st_active) {
            int flags = st_flags & ~(kFlagRestart | kFlagHold);
            cs.rr[j] = t;
            cs.qp[j] = tot[NV - 1];
            cs.rr_ref[j] = t;
            // a restarted direction is the residual itself (no previous one).
            // BF16 storage keeps its directions in index order; in even-odd
            // order, where a drop takes half as many steps, the kept ones cost
            // more than they bring (8^4 x 3, 1e-8, an FP64-emulated run: 29.8
            // steps kept, 26.1 restarted at drop 0.002; 28.7 and 21.3 at 0.01)
            if ((st_flags & kFlagRestart) || cs.ru_restart) cs.beta[j] = 0.0;
            if (t <= cs.tol2 * st_bb) {
                cs.active[j] = 0;
                flags |= kFlagConverged;
            }
            cs.flags[j] = flags;
        }
    } else if (EPI == kEpiStats || EPI == kEpiStatsP1) {
        cs.true_rr[j] = t;
    } else {
        cs.tj[2 * j] = tot[0];
        cs.tj[2 * j + 1] = NV > 1 ? tot[NV - 1] : 0.0;
    }
}

template <int NV, int EPI>
__global__ __launch_bounds__(kBlock) void k_finish(Red rd, CgState cs) {
    k_finish_body<NV, EPI>(blockIdx.x, rd, cs);
}

// Finishing kernel of a CG iteration (single reduction), one workgroup per
// lane.  From the stencil's partials, pq = Re p^H q and qq = |q|^2 (q = A p
// as stored; with BF16 storage also rq = Re r^H q and rp = Re r^H p), and
// from the last update's, rr = |r|^2 (the residual as stored) and
// Re q_prev^H p:
//   FP64: a lane with rr <= tol^2 |b|^2 stops (converged);
//   BF16: a lane whose rr fell below delta^2 times its value at the last
//         reliable update holds (does not move) until that update;
//   alpha = rr / pq (BF16: rp / pq),
//   |r - alpha q|^2 = rr - 2 alpha rq + alpha^2 qq   (the new residual's
//         norm, known before the update that forms it; rq as below),
//   beta = |r - alpha q|^2 / rr,
// so that one kernel can then form x, r and p (the new |r|^2 is also summed
// there, exactly, for the next iteration: the expansion's cancellation
// never carries over from one iteration to the next).  pq <= 0: FP64 stops
// the lane (breakdown); mixed precision flags it to restart its direction
// at the next reliable update (FP32 takes a steepest-descent step
// meanwhile, BF16 holds).
// The lane's state as the finishing kernel reads it (loaded before the
// partials, so that the two latencies overlap).
struct LaneState {
    double ref = 0.0, bb = 0.0, beta = 0.0;
    int active = 0, flags = 0, iters = 0;
};

__device__ __forceinline__ LaneState load_lane_state(int j, const CgState &cs) {
    LaneState st;
    st.ref = cs.rr_ref[j];
    st.bb = cs.bb[j];
    st.beta = cs.beta[j];
    st.active = cs.active[j];
    st.flags = cs.flags[j];
    st.iters = cs.iters[j];
    return st;
}

__device__ __forceinline__ void finish_cg_epilogue(int j, const CgState &cs, const LaneState &ls, const double (&d3)[4],
                                                   const double (&d2)[2]);

__device__ __forceinline__ void k_finish_cg_body(int lane, const Red &rd, const CgState &cs) {
    __shared__ double sm[6 * kBlock / 64];
    const int tid = threadIdx.x;
    LaneState ls;
    if (tid == 0) ls = load_lane_state(lane, cs);
    double d3[4], d2[2];
    lane_totals<4, 2>(rd.part1 + (size_t)lane * rd.nblk * 4, rd.part2 + (size_t)lane * rd.nblk * 2, rd.nblk, d3, d2, sm);
    if (tid == 0) finish_cg_epilogue(lane, cs, ls, d3, d2);
}

// The same with one wavefront per lane (the multi-instance engine: a few
// dozen partials per lane).
__device__ __forceinline__ void k_finish_cg_wave_body(int lane, const Red &rd, const CgState &cs) {
    LaneState ls;
    if ((threadIdx.x & 63) == 0) ls = load_lane_state(lane, cs);
    double d3[4], d2[2];
    lane_total_wave<4>(rd.part1 + (size_t)lane * rd.nblk * 4, rd.nblk, d3);
    lane_total_wave<2>(rd.part2 + (size_t)lane * rd.nblk * 2, rd.nblk, d2);
    if ((threadIdx.x & 63) == 0) finish_cg_epilogue(lane, cs, ls, d3, d2);
}

// An FP32 lane whose |r|^2 has grown this far above its last true residual's (CG's
// own residual may rise by the root of the condition number in norm), or is not
// finite, has lost its directions: where a Krylov space is exhausted (a small
// lattice, a few plane waves) the recursion falls far below what FP32 resolves
// and what follows is noise that grows.  It restarts at the next reliable update.
constexpr double kDiverged = 1e6;

// alpha, beta, flags and counts of lane j from its totals (thread-local)
__device__ __forceinline__ void finish_cg_epilogue(int j, const CgState &cs, const LaneState &ls, const double (&d3)[4],
                                                   const double (&d2)[2]) {
    const double st_ref = ls.ref, st_bb = ls.bb, st_beta = ls.beta;
    const int st_active = ls.active, st_flags = ls.flags, st_iters = ls.iters;
    const double rr = d2[0], pq = d3[0], qq = d3[2];
    // r^H q: since the residual is r = p - beta p_prev (beta the one that
    // formed p), r^H q = p^H q - beta p_prev^H A p, and p_prev^H A p =
    // (A p_prev)^H p = q_prev^H p was summed by the update that formed p (A
    // Hermitian; no conjugacy assumed).  A reliable update replaces r by the
    // true residual and keeps p, so the relation then holds up to the drift
    // of the recursive residual, which with FP32 storage is a few 1e-5 of
    // |r| and with BF16 storage up to about a tenth: there (rq_direct) the
    // stencil sums r^H q itself, and also r^H p, so that alpha is the exact
    // line search along p, Re r^H p / p^H A p, instead of |r|^2 / p^H A p
    // (equal while r^H p_prev = 0; after a replacement the first step
    // restores that orthogonality).
    const double rq = cs.rq_direct ? d3[1] : pq - st_beta * d2[1];
    const double rp = cs.rq_direct ? d3[3] : rr;
    int active = st_active, flags = st_flags, iters = st_iters;
    // a held lane keeps its direction, and with it the beta that formed it
    double alpha = 0.0, beta = st_beta;
    if (active) {
        if (cs.exact && rr <= cs.tol2 * st_bb) {
            active = 0;
            flags |= kFlagConverged;
        } else if (cs.hold && !(rr >= cs.delta2 * st_ref)) {
            flags |= kFlagHold;  // due a reliable update (or not finite)
        } else if (!cs.exact && !cs.hold && !(rr <= kDiverged * st_ref)) {
            flags |= kFlagRestart;
        }
    }
    if (!active) beta = 0.0;
    if (active && !(flags & kFlagHold)) {
        if (!(pq > 0.0) || !isfinite(pq)) {
            beta = 0.0;
            if (cs.exact) {
                flags |= kFlagBreakdown;
                active = 0;
            } else {
                flags |= kFlagRestart | (cs.hold ? kFlagHold : 0);
            }
        } else {
            alpha = rp / pq;
            const double rn = rr - 2.0 * alpha * rq + alpha * alpha * qq;
            beta = rn > 0.0 && isfinite(rn) ? rn / rr : 0.0;
            ++iters;
        }
    }
    cs.rr[j] = rr;
    cs.qp[j] = d2[1];
    cs.alpha[j] = alpha;
    cs.beta[j] = beta;
    cs.active[j] = active;
    cs.flags[j] = flags;
    cs.iters[j] = iters;
}

__global__ __launch_bounds__(kBlock) void k_finish_cg(Red rd, CgState cs) { k_finish_cg_body(blockIdx.x, rd, cs); }

// Control word for the host: [0] active lanes, [1] active lanes whose
// recursive residual meets tol, [2] active lanes due a reliable update,
// [3] lanes that broke down; ctrld[0] the largest |r|^2 / (tol^2 |b|^2) of
// an active lane (how far the slowest one still is from convergence);
// ctrld[1] (mixed precision) the smallest |r|^2 / (delta^2 |r_ref|^2) of an
// active lane not yet due a reliable update (how close the next one is;
// 0 if there is none).
// One wavefront; the counts and extremes of its threads meet by butterflies
// (with one thread reading 64 of each from LDS the launch took 7.1 us, now 2.4).
__device__ __forceinline__ void k_ctrl_body(const CgState &cs, int W) {
    const int t = threadIdx.x;
    int na = 0, nk = 0, nru = 0, nb = 0;
    double wr = 0.0, fr = HUGE_VAL;
    for (int k = t; k < W; k += 64) {
        const double rr = cs.rr[k], ref = cs.rr_ref[k], bb = cs.bb[k];
        const int flags = cs.flags[k];
        nb += (flags & kFlagBreakdown) ? 1 : 0;
        if (!cs.active[k]) continue;
        ++na;
        const double goal = cs.tol2 * bb;
        if (rr <= goal) ++nk;
        const bool due = !(rr >= cs.delta2 * ref) || (flags & (kFlagRestart | kFlagHold));
        if (due)
            ++nru;
        else if (!cs.exact)
            fr = fmin(fr, rr / (cs.delta2 * ref));
        wr = fmax(wr, rr / goal);
    }
    for (int off = 32; off > 0; off >>= 1) {
        na += __shfl_xor(na, off, 64);
        nk += __shfl_xor(nk, off, 64);
        nru += __shfl_xor(nru, off, 64);
        nb += __shfl_xor(nb, off, 64);
        wr = fmax(wr, __shfl_xor(wr, off, 64));
        fr = fmin(fr, __shfl_xor(fr, off, 64));
    }
    if (t != 0) return;
    cs.ctrl[0] = na;
    cs.ctrl[1] = nk;
    cs.ctrl[2] = nru;
    cs.ctrl[3] = nb;
    cs.ctrld[0] = wr;
    cs.ctrld[1] = isfinite(fr) ? fr : 0.0;
    if (cs.live) *cs.live = na;
}

__global__ void k_ctrl(CgState cs, int W) { k_ctrl_body(cs, W); }

// ============================================================ kernels

// The operator's device tables in one pass over the hop-link elements
// e = ((site * 8 + dir) * nc + a) * nc + b: the neighbour table nbr[site][8]
// (x + mu for dir = mu < 4, then x - mu; written by the elements a = b = 0),
// the FP64 links [N][4][nc][nc] (from the forward elements; if u64), and
// the hop links [N][8][nc][nc], entry (x, mu) = U_mu(x) and (x, 4 + mu) =
// U_mu(x - mu) (not conjugated), in the storage LS (if u8) and in FP64 (if
// u8x), so that a site's eight hops are one contiguous record.  The ABI links
// are complex128 [4][N][nc][nc]; without links (abi null) only the
// neighbour table.
template <typename LS>
__global__ void k_prepare(Lat L, int nc, const double2 *__restrict__ abi, int *__restrict__ nbr,
                          double2 *__restrict__ u64, LS *__restrict__ u8, double2 *__restrict__ u8x) {
    const int ne = abi ? nc * nc : 1;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= 8LL * L.N * ne) return;
    const int ab = (int)(e % ne);
    const long long t = e / ne;
    const int dir = (int)(t % 8), s = (int)(t / 8), site = lex_of(L, s), mu = dir & 3;
    int r = site, x = 0, stride = 1;
    for (int d = 3; d >= mu; --d) {
        if (d == mu) x = r % L.D[d];
        else stride *= L.D[d];
        r /= L.D[d];
    }
    const int y = dir < 4 ? site + (x + 1 == L.D[mu] ? -(L.D[mu] - 1) : 1) * stride
                          : site + (x == 0 ? L.D[mu] - 1 : -1) * stride;
    if (ab == 0) stg(nbr + (size_t)s * 8 + dir, site_of(L, y));
    if (!abi) return;
    const double2 v = ldg(abi + ((size_t)mu * L.N + (dir < 4 ? site : y)) * nc * nc + ab);
    if (u8) St<LS>::st(u8, e, (typename St<LS>::R)v.x, (typename St<LS>::R)v.y);
    if (u8x) stg(u8x + e, v);
    if (u64 && dir < 4) stg(u64 + ((size_t)s * 4 + mu) * nc * nc + ab, v);
}

// Initialise one block of W right-hand sides: r = p = b (storage precision),
// xlo = 0 (x64 is the first fold's to write), and |b|^2 per lane; the finishing
// workgroup sets up the CG scalars.
// SRC 0: probes generated from ProbeGen (whoever needs b again regenerates
// it; index order, k_init_probe below in even-odd order); 1: from ABI b; 2: from an FP64 block src in index order; these two
// also write b (FP64).  In even-odd order the odd half of p is -b / c, from
// which the stencil that follows (kStInit) forms r = p = b_e + H b_o / c.
template <typename S, int SRC>
__device__ __forceinline__ void k_init_body(const Blk &bk, Launch L, ProbeGen g, const double2 *babi, long long rhs0,
                                            long long nvalid, double2 *b64, S *__restrict__ r, S *__restrict__ p,
                                            S *__restrict__ xlo, double hop_scale, Red rd) {
    __shared__ double sm[2 * kBlock];
    const int tid = threadIdx.x, W = L.W, logW = L.logW;
    const int j = tid & (W - 1);
    const int nc = L.nc;
    const unsigned long long seedmix = SRC == 0 ? mix64(g.seed) : 0ull;
    const ProbeLane pl = SRC == 0 ? probe_lane(g, nc, g.rhs0 + j) : ProbeLane{};
    double acc[2] = {0.0, 0.0};  // |b|^2, and 0 for q^H p (no previous direction)
    int t0, t1;
    tile_range(bk, full_tiles(L), t0, t1);
    for (int t = t0; t < t1; ++t) {
        const int site = t * (kBlock >> logW) + (tid >> logW);
        if (site >= L.lat.N) continue;
        const int x = lex_of(L.lat, site);
        const bool odd = site >= L.ns;  // (even-odd order only)
        const double f = odd ? -hop_scale : 1.0;
        for (int a = 0; a < nc; ++a) {
            double re = 0.0, im = 0.0;
            const size_t i = ((size_t)(site * nc + a) << logW) + j;
            if (SRC == 0) {
                if (j < g.nvalid) probe_at(g, seedmix, L.lat, nc, pl, x, a, re, im);
            } else if (SRC == 1) {
                if (j < nvalid) {
                    const double2 v = babi[((size_t)(rhs0 + j) * L.lat.N + x) * nc + a];
                    re = v.x;
                    im = v.y;
                }
            } else {
                const double2 v = babi[((size_t)(x * nc + a) << logW) + j];
                re = v.x;
                im = v.y;
            }
            if (SRC != 0) b64[i] = make_double2(re, im);
            St<S>::st(p, i, (typename St<S>::R)(f * re), (typename St<S>::R)(f * im));
            acc[0] += re * re + im * im;
            if (odd) continue;
            if (!L.lat.eo) St<S>::st(r, i, (typename St<S>::R)re, (typename St<S>::R)im);
            St<S>::st(xlo, i, 0, 0);
        }
    }
    block_partials_to<2>(bk, acc, W, logW, rd.part2, rd.nblk, sm);
}

template <typename S, int SRC>
__global__ __launch_bounds__(kBlock) void k_init(Launch L, ProbeGen g, const double2 *babi, long long rhs0,
                                                 long long nvalid, double2 *b64, S *__restrict__ r, S *__restrict__ p,
                                                 S *__restrict__ xlo, double hop_scale, Red rd) {
    k_init_body<S, SRC>(own_blk(), L, g, babi, rhs0, nvalid, b64, r, p, xlo, hop_scale, rd);
}

// Even-odd order, probes: the whole start of a block in one pass,
// r = p_e = b_e + H b_o / c with |b|^2 and |r|^2 per lane.  A probe is nonzero
// on the sites of one colour only, so a thread generates the values of its
// site's neighbours itself where they are nonzero, and multiplies only those
// by their links (FP64): the pass writes its vectors and reads next to
// nothing, where writing b and x64 and then applying the hopping term to b
// moved four times as much (16^4 x 3, FP32, W = 64, 960 colours: 184 us for
// the two passes, 50 us in one; 16 colours, BF16: 200 and about 120).
// The neighbours' indices and colours are found once per site, by the whole
// workgroup for a stretch of sites at a time (the index order takes several
// integer divisions, which the W lanes of a site would all repeat).  The odd
// half of p is the first step's to write, x64 the first fold's.
template <typename S, int NC, bool LINKS>
__device__ __forceinline__ void k_init_probe_body(const Blk &bk, const Launch &L, const ProbeGen &g,
                                                  S *__restrict__ r, S *__restrict__ p, S *__restrict__ xlo,
                                                  double hop_scale, const double2 *__restrict__ U, const Red &rd) {
    constexpr int kStretch = 32;  // sites at a time (W < 8: one tile's)
    __shared__ double sm[4 * kBlock];
    __shared__ int sx[10 * kBlock], sc[10 * kBlock];  // [neighbour][site]: ABI index (displaced) and colour
    const int tid = threadIdx.x, W = L.W, logW = L.logW;
    const int j = tid & (W - 1), spt = kBlock >> logW;
    const int nst = max(kStretch, spt);
    const Lat &lat = L.lat;
    const unsigned long long seedmix = mix64(g.seed);
    const ProbeLane pl = probe_lane(g, NC, g.rhs0 + j);
    const bool valid = j < g.nvalid;
    // the noise counter of site 0, component 0 (see noise), and |b|^2 of a lit site
    const unsigned long long ctr0 = (unsigned long long)pl.s * (unsigned long long)lat.N * NC;
    const double bsite = (g.noise == DP_NOISE_Z2_COMPLEX ? 2.0 : 1.0) * (g.dilute ? 1 : NC);
    double bb[2] = {0.0, 0.0}, acc[4] = {0.0, 0.0, 0.0, 0.0};
    int t0, t1;
    tile_range(bk, L.ntiles, t0, t1);
    const int end = min(t1 * spt, L.ns);
    for (int s0 = t0 * spt; s0 < end; s0 += nst) {
        __syncthreads();
        for (int k = tid; k < nst && s0 + k < end; k += kBlock) {
            // the site's coordinates, moved by the probes' displacement; the
            // neighbours', and the odd site of the same internal index (mate)
            int x = lex_of(lat, s0 + k);
            if (g.shift) x = shift0(lat, x, -g.shift);
            int rem = x, st = 1;
#pragma unroll
            for (int d = 3; d >= 0; --d) {
                const int D = lat.D[d], q = rem / D, c = rem - q * D;
                sx[d * nst + k] = x + (c + 1 == D ? 1 - D : 1) * st;
                sx[(d + 4) * nst + k] = x + (c == 0 ? D - 1 : -1) * st;
                rem = q;
                st *= D;
            }
            sx[8 * nst + k] = x;
            sx[9 * nst + k] = x ^ 1;
#pragma unroll
            for (int d = 0; d < 10; ++d) sc[d * nst + k] = ldg(g.colors + sx[d * nst + k]);
        }
        __syncthreads();
        for (int k = tid >> logW; k < nst && s0 + k < end; k += spt) {
            const int site = s0 + k;
            double ar[NC] = {}, ai[NC] = {};
            // the hop from neighbour dir of the probe's component b
            auto hop = [&](int dir, int y, int b) {
                double vr, vi;
                noise_at(seedmix, ctr0 + (unsigned)(y * NC + b), g.noise, vr, vi);
                const double2 *u = U + ((size_t)site * 8 + dir) * NC * NC;
#pragma unroll
                for (int a = 0; a < NC; ++a) {
                    double2 w = make_double2(a == b ? 1.0 : 0.0, 0.0);
                    if (LINKS) w = ldg(u + (dir < 4 ? a * NC + b : b * NC + a));
                    if (dir >= 4) w.y = -w.y;
                    ar[a] = fma(w.x, vr, fma(-w.y, vi, ar[a]));
                    ai[a] = fma(w.x, vi, fma(w.y, vr, ai[a]));
                }
            };
#pragma unroll
            for (int dir = 0; dir < 8; ++dir) {
                if (!valid || sc[dir * nst + k] != pl.c) continue;
                const int y = sx[dir * nst + k];
                if (g.dilute) {
                    hop(dir, y, pl.a);
                } else {
#pragma unroll
                    for (int b = 0; b < NC; ++b) hop(dir, y, b);
                }
            }
            const bool own = valid && sc[8 * nst + k] == pl.c, mate = valid && sc[9 * nst + k] == pl.c;
            bb[0] += ((own ? 1.0 : 0.0) + (mate ? 1.0 : 0.0)) * bsite;
            const unsigned long long ctr = ctr0 + (unsigned)(sx[8 * nst + k] * NC);
#pragma unroll
            for (int a = 0; a < NC; ++a) {
                double br = 0.0, bi = 0.0;
                if (own && !(g.dilute && a != pl.a)) noise_at(seedmix, ctr + a, g.noise, br, bi);
                const size_t i = ((size_t)(site * NC + a) << logW) + j;
                typename St<S>::R rr = (typename St<S>::R)fma(hop_scale, ar[a], br);
                typename St<S>::R ri = (typename St<S>::R)fma(hop_scale, ai[a], bi);
                St<S>::st(r, i, rr, ri);
                St<S>::st(p, i, rr, ri);
                St<S>::st(xlo, i, 0, 0);
                St<S>::round(rr, ri);
                acc[2] += (double)rr * rr + (double)ri * ri;
            }
        }
    }
    block_partials_to<2>(bk, bb, W, logW, rd.part2, rd.nblk, sm);
    __syncthreads();
    block_partials<4>(bk, acc, W, logW, rd, sm);
}

template <typename S, int NC, bool LINKS>
__global__ __launch_bounds__(kBlock) void k_init_probe(Launch L, ProbeGen g, S *__restrict__ r, S *__restrict__ p,
                                                       S *__restrict__ xlo, double hop_scale,
                                                       const double2 *__restrict__ U, Red rd) {
    k_init_probe_body<S, NC, LINKS>(own_blk(), L, g, r, p, xlo, hop_scale, U, rd);
}

// the probes of g in FP64, index order [site][nc][W]
__global__ __launch_bounds__(kBlock) void k_probe_fill(Launch L, ProbeGen g, double2 *__restrict__ out) {
    const int j = threadIdx.x & (L.W - 1);
    const unsigned long long seedmix = mix64(g.seed);
    const ProbeLane pl = probe_lane(g, L.nc, g.rhs0 + j);
    const int spt = kBlock >> L.logW;
    for (int x = (int)blockIdx.x * spt + (int)(threadIdx.x >> L.logW); x < L.lat.N; x += (int)gridDim.x * spt)
        for (int a = 0; a < L.nc; ++a) {
            double re = 0.0, im = 0.0;
            if (j < g.nvalid) probe_at(g, seedmix, L.lat, L.nc, pl, x, a, re, im);
            stg(out + ((size_t)(x * L.nc + a) << L.logW) + j, make_double2(re, im));
        }
}

// q = A p for one block of right-hand sides; with CG, also p^H q per lane
// and the other dot products of a CG iteration (k_finish_cg).
// STAGE: links of the tile's sites staged in LDS (W >= 16).
// ------------------------------------------------------------ stencil helpers

__device__ __forceinline__ float fmaR(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double fmaR(double a, double b, double c) { return fma(a, b, c); }

// Element i of a block vector, addressed by a 32-bit byte offset from the
// vector's base: with the base uniform (a kernel argument, or read from a
// slot descriptor by the whole workgroup) the access takes the scalar-base +
// 32-bit-offset form, with no 64-bit address arithmetic per element.  Every
// block vector of the stencil kernels is smaller than 4 GiB (the host
// rejects wider blocks).
template <typename T>
__device__ __forceinline__ const T *at32(const T *base, unsigned i) {
    return (const T *)((const char *)base + i * (unsigned)sizeof(T));
}
template <typename T>
__device__ __forceinline__ T *at32(T *base, unsigned i) {
    return (T *)((char *)base + i * (unsigned)sizeof(T));
}

// p as an opaque uniform value (p must be the same in every thread of the
// wavefront): the compiler cannot then fold a colour row's offset into
// per-thread 64-bit address arithmetic, and every load of a site's colours
// shares the one 32-bit site offset, each from its own scalar base.
template <typename T>
__device__ __forceinline__ T *ubase(T *p) {
    const unsigned long long a = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)a);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(a >> 32));
    return (T *)(((unsigned long long)hi << 32) | lo);
}

// The colour-row bases v + b * W (b < NC) of a block vector.
template <typename T, int NC>
struct Rows {
    T *b[NC];
    __device__ __forceinline__ Rows(T *v, int logW) {
#pragma unroll
        for (int c = 0; c < NC; ++c) b[c] = ubase(v + ((size_t)c << logW));
    }
};

// element (site y, colour b, lane j) of a block vector
__device__ __forceinline__ unsigned vidx(int y, int nc, int b, int logW, int j) {
    return ((unsigned)(y * nc + b) << logW) + (unsigned)j;
}

// colour components of lane j at site y
template <typename S, int NC>
__device__ __forceinline__ void ld_site(const S *__restrict__ v, int y, int logW, int j,
                                        typename St<S>::R (&re)[NC], typename St<S>::R (&im)[NC]) {
    const S *row = v + ((size_t)(y * NC) << logW);
#pragma unroll
    for (int b = 0; b < NC; ++b) St<S>::ld(row, (unsigned)((b << logW) + j), re[b], im[b]);
}

// the same from colour-row bases, through one 32-bit site offset
template <typename S, int NC>
__device__ __forceinline__ void ld_rows(const Rows<const S, NC> &v, int y, int logW, int j,
                                        typename St<S>::R (&re)[NC], typename St<S>::R (&im)[NC]) {
    const unsigned i = vidx(y, NC, 0, logW, j);
#pragma unroll
    for (int b = 0; b < NC; ++b) St<S>::ld(at32(v.b[b], i), 0, re[b], im[b]);
}

// and stores colour components to colour-row bases
template <typename S, int NC>
__device__ __forceinline__ void st_rows(const Rows<S, NC> &v, int y, int logW, int j, int b,
                                        typename St<S>::R re, typename St<S>::R im) {
    St<S>::st(at32(v.b[b], vidx(y, NC, 0, logW, j)), 0, re, im);
}

// acc -= U v (DAG = false) or acc -= U^H v (DAG = true), u = 3x3 (or 1x1)
// complex matrix as (re, im) pairs in row-major order; four FMAs per
// complex multiply-subtract.
template <typename R, int NC, bool DAG>
__device__ __forceinline__ void mul_sub(const R *u, const R (&vr)[NC], const R (&vi)[NC], R (&ar)[NC], R (&ai)[NC]) {
#pragma unroll
    for (int a = 0; a < NC; ++a) {
#pragma unroll
        for (int b = 0; b < NC; ++b) {
            const int e = DAG ? b * NC + a : a * NC + b;
            const R ur = u[2 * e];
            const R ui = DAG ? -u[2 * e + 1] : u[2 * e + 1];
            ar[a] = fmaR(-ur, vr[b], ar[a]);
            ar[a] = fmaR(ui, vi[b], ar[a]);
            ai[a] = fmaR(-ur, vi[b], ai[a]);
            ai[a] = fmaR(-ui, vr[b], ai[a]);
        }
    }
}

// Stages the neighbour indices of the tile's sites in LDS (the bodies
// without links).  All threads of the workgroup call it; it ends with a
// barrier.
__device__ __forceinline__ void stage_nbr(int *snb, const SiteWalk &wk, int item0, int sites_per_tile,
                                          const int *__restrict__ nbr) {
    const int tid = threadIdx.x;
    __syncthreads();
    for (int e = tid; e < sites_per_tile * 8; e += kBlock)
        snb[e] = item0 + e / 8 < wk.items ? ldg(nbr + walk_site(wk, item0 + e / 8) * 8 + (e & 7)) : 0;
    __syncthreads();
}

// The packed products of one hop on bf16x2 words (low half real, high
// half imaginary), from the stored link word w = (Ur, Ui) and the vector
// word v = (vr, vi): re += dot(w, c1), im += dot(w, c2).  Forward hop
// (U v): c1 = (vr, -vi), c2 = (vi, vr).  Backward hop (U^H v, element (a, b)
// taken from U[b][a]): c1 = v, c2 = (vi, -vr).  The two words are formed once
// per vector word and used for the NC link elements that multiply it; the
// products are those of the complex multiplication, exactly.
__device__ __forceinline__ void hop_vec_words(uint32_t v, bool dag, uint32_t &c1, uint32_t &c2) {
    const uint32_t sw = (v >> 16) | (v << 16);  // (vi, vr)
    c1 = dag ? v : v ^ 0x80000000u;
    c2 = dag ? sw ^ 0x80000000u : sw;
}

// Orders this wavefront's LDS accesses before the call against those after
// it (LDS operations of one wavefront complete in issue order; the fences
// keep the compiler from moving accesses across).
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The tile items a wavefront stages and works on: n items from `first` (in
// the tile) into LDS slots from slot0.  With W <= 64 a wavefront holds 64 / W
// whole lane groups of G items each; with W > 64 a lane group spans W / 64
// wavefronts, which stage a copy each.  slot: the slot of member 0 of this
// thread's lane group.
struct WaveItems {
    int first, n, slot0, slot;
};

__device__ __forceinline__ WaveItems wave_items(int logW, int G) {
    const int tid = threadIdx.x, wv = tid >> 6, sl = tid >> logW;
    WaveItems w;
    if (logW <= 6) {
        w.n = G << (6 - logW);
        w.first = wv * w.n;
        w.slot0 = w.first;
        w.slot = G * sl;
    } else {
        w.n = G;
        w.first = G * sl;
        w.slot0 = wv * G;
        w.slot = w.slot0;
    }
    return w;
}

// Stages the hop links (converted to R) and neighbour indices of the
// wavefront's items item0 + wi.first .. + wi.n - 1 into its LDS slots, by
// that wavefront alone: each wavefront stages what its own threads read, so
// the tile loop takes no workgroup barrier.  Where the LDS layout is the
// memory layout (FP32 and FP64 links) the copy moves 16 bytes per thread.
template <typename LS, typename R, int NC, bool LINKS>
__device__ __forceinline__ void stage_hops_wave(R *su, int *snb, const SiteWalk &wk, int item0, const WaveItems &wi,
                                                const LS *__restrict__ U8, const int *__restrict__ nbr) {
    const int lane = threadIdx.x & 63;
    constexpr int kE = 8 * NC * NC;  // complex link elements of a site
    const int first = item0 + wi.first, n = wi.n;
    wave_fence();  // this wavefront's reads of the previous tile come first
    if (LINKS) {
        if constexpr (sizeof(LS) == 2 * sizeof(R)) {
            constexpr int kV = kE * (int)sizeof(LS) / 16;
            for (int e = lane; e < n * kV; e += 64) {
                const int i = e / kV, k = e - i * kV;
                uint4 v = make_uint4(0u, 0u, 0u, 0u);
                if (first + i < wk.items) v = ldg((const uint4 *)(U8 + (size_t)walk_site(wk, first + i) * kE) + k);
                ((uint4 *)(su + (size_t)(wi.slot0 + i) * kE * 2))[k] = v;
            }
        } else {
            for (int e = lane; e < n * kE; e += 64) {
                const int i = e / kE, k = e - i * kE;
                typename St<LS>::R re = 0, im = 0;
                if (first + i < wk.items) St<LS>::ld(U8, (size_t)walk_site(wk, first + i) * kE + k, re, im);
                su[((size_t)(wi.slot0 + i) * kE + k) * 2] = (R)re;
                su[((size_t)(wi.slot0 + i) * kE + k) * 2 + 1] = (R)im;
            }
        }
    }
    for (int e = lane; e < n * 8; e += 64)
        snb[wi.slot0 * 8 + e] = first + e / 8 < wk.items ? ldg(nbr + walk_site(wk, first + e / 8) * 8 + (e & 7)) : 0;
    wave_fence();
}

// Starts the copy of one tile's hop links (as stored, [site][dir][a][b]) and
// neighbour indices into an LDS buffer laid out the same way: the links of
// the tile's sites, then their [site][8] indices.  16-byte loads that write
// LDS directly, without registers, issued by every wavefront for its share
// of the tile.  The copy is complete for this wavefront after its next
// `s_waitcnt vmcnt(0)`, for the workgroup after the barrier that follows it.
// Sites past the walk's end copy site 0 (their values are not used).
template <typename LS, int NC>
__device__ __forceinline__ void dma_tile(void *buf, const SiteWalk &wk, int item0, int sites_per_tile,
                                         const LS *__restrict__ U, const int *__restrict__ nbr) {
    constexpr int kSiteB = 8 * NC * NC * (int)sizeof(LS);  // bytes of a site's hop links
    static_assert(kSiteB % 16 == 0, "a site's hop links are whole 16-byte pieces");
    constexpr int kLC = kSiteB / 16;
    const int nlc = sites_per_tile * kLC, nch = nlc + sites_per_tile * 2;
    const int lane = threadIdx.x & 63;
    for (int c0 = (threadIdx.x >> 6) * 64; c0 < nch; c0 += kBlock) {
        const int c = c0 + lane;
        if (c >= nch) continue;
        const bool link = c < nlc;
        const int s_l = link ? c / kLC : (c - nlc) >> 1;
        const int k = link ? c - s_l * kLC : (c - nlc) & 1;
        const int site = item0 + s_l < wk.items ? walk_site(wk, item0 + s_l) : 0;
        const char *src = link ? (const char *)U + (size_t)site * kSiteB + 16 * k
                               : (const char *)(nbr + (size_t)site * 8) + 16 * k;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                         (__attribute__((address_space(3))) void *)((char *)buf + 16 * c0), 16, 0, 0);
    }
}

// dma_tile with the division of the pieces among the threads taken once:
// thread (wavefront w, lane) copies pieces 64 (w + 4 i) + lane, i < kN, of
// every tile, whose place in a site (piece of its links, or of its
// indices) does not change from tile to tile.
template <typename LS, int NC, int kN>
struct DmaPlan {
    static constexpr int kSiteB = 8 * NC * NC * (int)sizeof(LS);
    static constexpr int kLC = kSiteB / 16;
    int nch;          // pieces of a tile
    int s_l[kN];      // the piece's site in the tile
    int boff[kN];     // its byte offset in the site's links, or -1 - offset in its indices
    __device__ __forceinline__ DmaPlan(int sites_per_tile) {
        static_assert(kSiteB % 16 == 0, "a site's hop links are whole 16-byte pieces");
        const int nlc = sites_per_tile * kLC;
        nch = nlc + sites_per_tile * 2;
        const int c1 = (threadIdx.x >> 6) * 64 + (threadIdx.x & 63);
#pragma unroll
        for (int i = 0; i < kN; ++i) {
            const int c = c1 + i * kBlock;
            const bool link = c < nlc;
            s_l[i] = link ? c / kLC : (c - nlc) >> 1;
            boff[i] = link ? 16 * (c - (c / kLC) * kLC) : -1 - 16 * ((c - nlc) & 1);
        }
    }
    __device__ __forceinline__ void copy(void *buf, const SiteWalk &wk, int item0, const LS *__restrict__ U,
                                         const int *__restrict__ nbr) const {
        const int c1 = (threadIdx.x >> 6) * 64 + (threadIdx.x & 63);
#pragma unroll
        for (int i = 0; i < kN; ++i) {
            const int c0 = (threadIdx.x >> 6) * 64 + i * kBlock;  // uniform in the wavefront
            if (c0 >= nch) break;
            if (c1 + i * kBlock >= nch) continue;
            const int site = item0 + s_l[i] < wk.items ? walk_site(wk, item0 + s_l[i]) : 0;
            const char *src = boff[i] >= 0 ? (const char *)U + (size_t)site * kSiteB + boff[i]
                                           : (const char *)(nbr + (size_t)site * 8) + (-1 - boff[i]);
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src,
                                             (__attribute__((address_space(3))) void *)((char *)buf + 16 * c0), 16, 0,
                                             0);
        }
    }
};

// Waits for this wavefront's outstanding vector memory operations (the LDS
// copies above among them), then for the workgroup.
__device__ __forceinline__ void dma_wait_barrier() {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0); expcnt, lgkmcnt not waited for
    __syncthreads();
}

// The stencil on BF16-stored vectors and links: every complex product of a
// hop is two packed bf16 dot products accumulated in FP32 (the loaded words
// are used as they are, no unpacking); the modes are those of the generic
// body below.
template <int NC, bool LINKS, int MODE, int KIND>
__device__ __forceinline__ void k_stencil_bf16_body(const Blk &bk, Launch L, float diag, const bf16x2 *pin,
                                                    const bf16x2 *__restrict__ rin, bf16x2 *q,
                                                    bf16x2 *q2, const bf16x2 *__restrict__ U,
                                                    const int *__restrict__ nbr, int cg, Red rd) {
    constexpr bool HOP = KIND == kStHop;
    constexpr bool INIT = KIND == kStInit;  // no residual yet: only |q|^2 is summed
    constexpr bool STAGE = MODE == 1 && LINKS;
    constexpr int kMaxSites = kBlock / 16;
    // STAGE: two tile buffers, each [site][8 NC^2] link words then [site][8]
    // neighbour indices; the next tile is copied into one while the other is
    // read
    constexpr int kBuf = kMaxSites * 8 * NC * NC + kMaxSites * 8;
    constexpr bool kReuse = STAGE && 2 * kBuf * sizeof(uint32_t) >= 4 * kBlock * sizeof(double);
    __shared__ __align__(16) uint32_t su[STAGE ? 2 * kBuf : 1];
    __shared__ int snb[MODE == 1 && !STAGE ? kMaxSites * 8 : 1];
    __shared__ double sm_own[kReuse ? 1 : 4 * kBlock];
    double *sm = kReuse ? (double *)su : sm_own;
    const int tid = threadIdx.x, logW = L.logW, W = L.W;
    const int j = tid & (W - 1);
    const int sl = MODE == 2 ? __builtin_amdgcn_readfirstlane(tid >> logW) : tid >> logW;
    const int sites_per_tile = kBlock >> logW;
    const Rows<const bf16x2, NC> P(pin, logW), Rr(rin ? rin : pin, logW);
    const Rows<bf16x2, NC> Q(q, logW), Q2(INIT ? q2 : q, logW);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const SiteWalk wk = site_walk(L, bk, HOP ? 1 : 0);
    // STAGE: the copy of the next tile is in flight while this tile is worked
    // on, so that a tile waits for one round trip to memory rather than two
    // (at most 16 sites of 8 NC^2 + 8 words: two pieces per thread)
    const DmaPlan<bf16x2, NC, 2> plan(sites_per_tile);
    if (STAGE && wk.first * sites_per_tile < wk.items) plan.copy(su, wk, wk.first * sites_per_tile, U, nbr);
    // q of a tile is stored at the start of the next one, after the wait for
    // that tile's copy: the wait (for every outstanding vector memory
    // operation) then does not wait for the stores too
    uint32_t qw[NC];
    unsigned qi = 0;
    bool qpend = false;
    auto store_q = [&]() {
        if (!qpend) return;
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            bf16x2 o;
            o.v = qw[a];
            stg(at32(Q.b[a], qi), o);
            if (INIT) stg(at32(Q2.b[a], qi), o);
        }
        qpend = false;
    };
    int cur = 0;
    for (int t = wk.first; t * sites_per_tile < wk.items; t += wk.stride, cur ^= 1) {
        const int item0 = t * sites_per_tile;
        const uint32_t *lw = su + cur * kBuf;                       // this tile's link words
        const int *tnb = (const int *)lw + sites_per_tile * 8 * NC * NC;  // and neighbour indices
        if (STAGE) {
            // this tile's copy is complete, and every wavefront is done with the other buffer
            dma_wait_barrier();
            store_q();
            const int next0 = (t + wk.stride) * sites_per_tile;
            if (next0 < wk.items) plan.copy(su + (cur ^ 1) * kBuf, wk, next0, U, nbr);
        } else {
            store_q();
            if (MODE == 1) stage_nbr(snb, wk, item0, sites_per_tile, nbr);
        }
        if (item0 + sl >= wk.items) continue;
        const int site = walk_site(wk, item0 + sl);
        int y[9];
        y[0] = site;
#pragma unroll
        for (int dir = 0; dir < 8; ++dir)
            y[dir + 1] = STAGE ? tnb[sl * 8 + dir] : (MODE == 1 ? snb[sl * 8 + dir] : ldg(nbr + site * 8 + dir));
        uint32_t v[9][NC];
#pragma unroll
        for (int k = HOP ? 1 : 0; k < 9; ++k) {
            const unsigned i = vidx(y[k], NC, 0, logW, j);
#pragma unroll
            for (int b = 0; b < NC; ++b) v[k][b] = ldg(at32(P.b[b], i)).v;
        }
        uint32_t rv[NC];  // the residual at the site (CG: r^H q and r^H p summed here)
        if (cg && !INIT) {
            const unsigned i = vidx(site, NC, 0, logW, j);
#pragma unroll
            for (int b = 0; b < NC; ++b) rv[b] = ldg(at32(Rr.b[b], i)).v;
        }
        float hr[NC], hi[NC];  // sum of the hops
#pragma unroll
        for (int a = 0; a < NC; ++a) hr[a] = hi[a] = 0.0f;
#pragma unroll
        for (int dir = 0; dir < 8; ++dir) {
#pragma unroll
            for (int b = 0; b < NC; ++b) {
                if (!LINKS) {
                    hr[b] += __uint_as_float(v[dir + 1][b] << 16);
                    hi[b] += __uint_as_float(v[dir + 1][b] & 0xffff0000u);
                    continue;
                }
                uint32_t c1, c2;
                hop_vec_words(v[dir + 1][b], dir >= 4, c1, c2);
#pragma unroll
                for (int a = 0; a < NC; ++a) {
                    const int el = dir < 4 ? a * NC + b : b * NC + a;
                    const uint32_t w = STAGE ? lw[(sl * 8 + dir) * NC * NC + el]
                                             : ldg(U + ((size_t)site * 8 + dir) * NC * NC + el).v;
                    hr[a] = dot2_bf16(w, c1, hr[a]);
                    hi[a] = dot2_bf16(w, c2, hi[a]);
                }
            }
        }
        float pqs = 0, rqs = 0, qqs = 0, rps = 0;
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            bf16x2 o;
            if (HOP) {
                qw[a] = pack_bf16(diag * hr[a], diag * hi[a]);
                continue;
            }
            const float pr = __uint_as_float(v[0][a] << 16), pi = __uint_as_float(v[0][a] & 0xffff0000u);
            const float ar = fmaf(diag, pr, -hr[a]), ai = fmaf(diag, pi, -hi[a]);
            o.v = pack_bf16(ar, ai);
            qw[a] = o.v;
            if (INIT) {
                qqs = dot2_bf16(o.v, o.v, qqs);
            } else if (cg) {
                // the real parts of the dot products of the stored words (the
                // rounded q): one packed dot each, the products exact in FP32
                pqs = dot2_bf16(v[0][a], o.v, pqs);
                qqs = dot2_bf16(o.v, o.v, qqs);
                rqs = dot2_bf16(rv[a], o.v, rqs);
                rps = dot2_bf16(rv[a], v[0][a], rps);
            }
        }
        qi = vidx(site, NC, 0, logW, j);
        qpend = true;
        acc[0] += (double)pqs;
        acc[1] += (double)rqs;
        acc[2] += (double)qqs;
        acc[3] += (double)rps;
    }
    store_q();
    if (HOP || !cg) return;
    if (kReuse) __syncthreads();  // every wavefront is done with the link tile
    block_partials<4>(bk, acc, W, logW, rd, sm);
}

// hop link dir of site from the hop-link array, converted to R
template <typename LS, typename R, int NC>
__device__ __forceinline__ void ld_hop(const LS *__restrict__ U8, int site, int dir, R *u) {
    const LS *base = U8 + ((size_t)site * 8 + dir) * NC * NC;
#pragma unroll
    for (int e = 0; e < NC * NC; ++e) {
        typename St<LS>::R re, im;
        St<LS>::ld(base, e, re, im);
        u[2 * e] = (R)re;
        u[2 * e + 1] = (R)im;
    }
}

// The stencil q = A p for one block of right-hand sides, with p^H q summed
// per lane when `cg` is set (the first kernel of a CG iteration).
//
// MODE 0 (W < 16): every lane loads its site's links itself (the lanes of a
// site read the same addresses); for W = 1 (FP64, FP32) MODE 5 instead
// splits a site over 32 threads (k_stencil_split_body).  MODE 1 (16 <= W < 64): the links of the
// tile's sites are staged in LDS once and shared by the W lanes.  MODE 2
// (W >= 64): a wavefront covers one site, so the site index is uniform and
// the links and neighbour indices come through scalar loads; no LDS and no
// barriers.  MODES 3 and 4 (16 <= W < 64 with even x0-slabs) are MODE 1
// with two or four neighbouring sites per thread (k_stencil_group_body).  In every mode the vector loads of the site and its eight
// neighbours are issued before any arithmetic, so they are in flight
// together.
// KIND (StKind): in even-odd order a launch covers one half, the even sites
// with the formula above or the odd sites with the scaled hop sum alone.  (p
// and q are one vector in a hop launch, which reads its even half and writes
// its odd one; in kStInit each even site is read by the thread that
// overwrites it.)
template <typename S, typename LS, int NC, bool LINKS, int MODE, int KIND>
__device__ __forceinline__ void k_stencil_body(const Blk &bk, Launch L, typename St<S>::R diag, const S *pin,
                                               const S *__restrict__ rin, S *q, S *q2, const LS *__restrict__ U,
                                               const int *__restrict__ nbr, int cg, Red rd) {
    if constexpr (std::is_same<S, bf16x2>::value) {
        k_stencil_bf16_body<NC, LINKS, MODE, KIND>(bk, L, diag, pin, rin, q, q2, U, nbr, cg, rd);
        return;
    }
    constexpr bool HOP = KIND == kStHop;
    constexpr bool INIT = KIND == kStInit;
    using R = typename St<S>::R;
    constexpr bool STAGE = MODE == 1 && LINKS;
    constexpr int kMaxSites = kBlock / 16;
    // the reduction at the end reuses the link tile when there is one
    constexpr bool kReuse = STAGE && kMaxSites * 8 * NC * NC * 2 * sizeof(R) >= 4 * kBlock * sizeof(double);
    __shared__ __align__(16) R su[STAGE ? kMaxSites * 8 * NC * NC * 2 : 1];
    __shared__ int snb[MODE == 1 ? kMaxSites * 8 : 1];
    __shared__ double sm_own[kReuse ? 1 : 4 * kBlock];
    double *sm = kReuse ? (double *)su : sm_own;
    const int tid = threadIdx.x, logW = L.logW, W = L.W;
    const int j = tid & (W - 1);
    const int sl = MODE == 2 ? __builtin_amdgcn_readfirstlane(tid >> logW) : tid >> logW;
    const int sites_per_tile = kBlock >> logW;
    const WaveItems wi = wave_items(logW, 1);
    const Rows<const S, NC> P(pin, logW);
    const Rows<S, NC> Q(q, logW), Q2(INIT ? q2 : q, logW);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const SiteWalk wk = site_walk(L, bk, HOP ? 1 : 0);
    for (int t = wk.first; t * sites_per_tile < wk.items; t += wk.stride) {
        const int item0 = t * sites_per_tile;
        if (MODE == 1) stage_hops_wave<LS, R, NC, LINKS>(su, snb, wk, item0, wi, U, nbr);
        if (item0 + sl >= wk.items) continue;
        const int site = walk_site(wk, item0 + sl);
        int y[9];
        y[0] = site;
#pragma unroll
        for (int dir = 0; dir < 8; ++dir) y[dir + 1] = MODE == 1 ? snb[wi.slot * 8 + dir] : ldg(nbr + site * 8 + dir);
        R vr[9][NC], vi[9][NC];
#pragma unroll
        for (int k = HOP ? 1 : 0; k < 9; ++k) ld_rows<S, NC>(P, y[k], logW, j, vr[k], vi[k]);
        R ar[NC], ai[NC];
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            ar[a] = HOP ? (R)0 : diag * vr[0][a];
            ai[a] = HOP ? (R)0 : diag * vi[0][a];
        }
#pragma unroll
        for (int dir = 0; dir < 8; ++dir) {
            if (!LINKS) {
#pragma unroll
                for (int a = 0; a < NC; ++a) {
                    ar[a] -= vr[dir + 1][a];
                    ai[a] -= vi[dir + 1][a];
                }
                continue;
            }
            R u[2 * NC * NC];
            if (STAGE) {
#pragma unroll
                for (int e = 0; e < 2 * NC * NC; ++e) u[e] = su[(wi.slot * 8 + dir) * NC * NC * 2 + e];
            } else {
                ld_hop<LS, R, NC>(U, site, dir, u);
            }
            if (dir < 4)
                mul_sub<R, NC, false>(u, vr[dir + 1], vi[dir + 1], ar, ai);
            else
                mul_sub<R, NC, true>(u, vr[dir + 1], vi[dir + 1], ar, ai);
        }
        R pqs = 0, qqs = 0;
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            if (HOP) {  // the hops were subtracted
                st_rows<S, NC>(Q, site, logW, j, a, -diag * ar[a], -diag * ai[a]);
                continue;
            }
            st_rows<S, NC>(Q, site, logW, j, a, ar[a], ai[a]);
            if (INIT) st_rows<S, NC>(Q2, site, logW, j, a, ar[a], ai[a]);
            if (cg) {
                if (!INIT) pqs = fmaR(vr[0][a], ar[a], fmaR(vi[0][a], ai[a], pqs));
                qqs = fmaR(ar[a], ar[a], fmaR(ai[a], ai[a], qqs));
            }
        }
        acc[0] += (double)pqs;
        acc[2] += (double)qqs;
    }
    if (HOP || !cg) return;
    if (kReuse) __syncthreads();  // every wavefront is done with the link tile
    block_partials<4>(bk, acc, W, logW, rd, sm);
}

// MODES 3 and 4: MODE 1 with G sites per thread that are each other's
// neighbours, so the shared neighbours are loaded once.  When every XCD's
// slab has an even number of x0-slices, the slab walk (x0 fastest) puts the
// x0-slices of a pair at consecutive items: with G = 2 a thread takes items
// 2i, 2i + 1, sites s and s + V3 (x0 neighbours): 16 site loads per pair
// instead of 18.  With two slices per slab and an even D3, items 4i .. 4i + 3
// are s, s + V3, s + 1, s + V3 + 1 (x0 and x3 neighbours; 4i / 2 is even,
// so x3 + 1 does not wrap): 28 loads per quad instead of 36.  16^4, FP32,
// W = 32: 45.1 us (G = 1), 41.6 (G = 2), 40.6 (G = 4).  With a multiple of
// four slices per slab (MODE 6, LINE), items 4i .. 4i + 3 are four
// consecutive x0-slices of one (x1, x2, x3): s + h V3, 30 loads per four
// sites instead of 32 with pairs.
template <int G, bool LINE>
__device__ __forceinline__ int group_nb(int h, int dir) {
    // the group member that is neighbour dir of member h, or -1
    if (LINE) return (dir == 0 && h < G - 1) ? h + 1 : (dir == 4 && h > 0) ? h - 1 : -1;
    if (G == 2) return (h == 0 && dir == 0) ? 1 : (h == 1 && dir == 4) ? 0 : -1;
    switch (h * 8 + dir) {
        case 0 * 8 + 0: return 1;
        case 0 * 8 + 3: return 2;
        case 1 * 8 + 4: return 0;
        case 1 * 8 + 3: return 3;
        case 2 * 8 + 0: return 3;
        case 2 * 8 + 7: return 0;
        case 3 * 8 + 4: return 2;
        case 3 * 8 + 7: return 1;
        default: return -1;
    }
}

template <typename S, typename LS, int NC, bool LINKS, int G, bool LINE = false>
__device__ __forceinline__ void k_stencil_group_body(const Blk &bk, Launch L, typename St<S>::R diag,
                                                     const S *__restrict__ pin, const S *__restrict__ rin,
                                                     S *__restrict__ q, const LS *__restrict__ U,
                                                     const int *__restrict__ nbr, int cg, Red rd) {
    using R = typename St<S>::R;
    // BF16 storage (FP32 arithmetic on the unpacked values here) sums r^H q
    // and r^H p itself, like the packed BF16 body
    constexpr bool kDirect = std::is_same<S, bf16x2>::value;
    // (pairs need W >= 16, quads and lines W >= 32: at most 32 items per tile)
    constexpr int kMaxItems = G == 2 ? 2 * (kBlock / 16) : 4 * (kBlock / 32);
    // the reduction at the end reuses the link tile when it is large enough
    constexpr bool kReuse = LINKS && kMaxItems * 8 * NC * NC * 2 * sizeof(R) >= 4 * kBlock * sizeof(double);
    __shared__ __align__(16) R su[LINKS ? kMaxItems * 8 * NC * NC * 2 : 1];
    __shared__ int snb[kMaxItems * 8];
    __shared__ double sm_own[kReuse ? 1 : 4 * kBlock];
    double *sm = kReuse ? (double *)su : sm_own;
    const int tid = threadIdx.x, logW = L.logW, W = L.W;
    const int j = tid & (W - 1);
    const int sl = tid >> logW;
    const int items_per_tile = G * (kBlock >> logW);
    const WaveItems wi = wave_items(logW, G);
    const Rows<const S, NC> P(pin, logW), Rr(kDirect && rin ? rin : pin, logW);
    const Rows<S, NC> Q(q, logW);
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    const SiteWalk wk = site_walk(L, bk);
    for (int t = wk.first; t * items_per_tile < wk.items; t += wk.stride) {
        const int item0 = t * items_per_tile;
        stage_hops_wave<LS, R, NC, LINKS>(su, snb, wk, item0, wi, U, nbr);
        if (item0 + G * sl >= wk.items) continue;
        const int s0 = walk_site(wk, item0 + G * sl);
        R vor[G][NC], voi[G][NC];  // the members' own vectors
#pragma unroll
        for (int h = 0; h < G; ++h)
            ld_rows<S, NC>(P, s0 + (LINE ? h * wk.V3 : (h & 1) * wk.V3 + (h >> 1)), logW, j, vor[h], voi[h]);
        R pqs = 0, qqs = 0, rqs = 0, rps = 0;
#pragma unroll
        for (int h = 0; h < G; ++h) {
            const int ls = wi.slot + h;
            const int site = s0 + (LINE ? h * wk.V3 : (h & 1) * wk.V3 + (h >> 1));
            R rr_[NC], ri_[NC];  // BF16 storage: the residual (r^H q, r^H p summed here)
            if (kDirect && cg) ld_rows<S, NC>(Rr, site, logW, j, rr_, ri_);
            R vr[8][NC], vi[8][NC];
#pragma unroll
            for (int dir = 0; dir < 8; ++dir) {
                const int m = group_nb<G, LINE>(h, dir);
                if (m >= 0) {
#pragma unroll
                    for (int b = 0; b < NC; ++b) {
                        vr[dir][b] = vor[m][b];
                        vi[dir][b] = voi[m][b];
                    }
                } else {
                    ld_rows<S, NC>(P, snb[ls * 8 + dir], logW, j, vr[dir], vi[dir]);
                }
            }
            R ar[NC], ai[NC];
#pragma unroll
            for (int a = 0; a < NC; ++a) {
                ar[a] = diag * vor[h][a];
                ai[a] = diag * voi[h][a];
            }
#pragma unroll
            for (int dir = 0; dir < 8; ++dir) {
                if (!LINKS) {
#pragma unroll
                    for (int a = 0; a < NC; ++a) {
                        ar[a] -= vr[dir][a];
                        ai[a] -= vi[dir][a];
                    }
                    continue;
                }
                R u[2 * NC * NC];
#pragma unroll
                for (int e = 0; e < 2 * NC * NC; ++e) u[e] = su[(ls * 8 + dir) * NC * NC * 2 + e];
                if (dir < 4)
                    mul_sub<R, NC, false>(u, vr[dir], vi[dir], ar, ai);
                else
                    mul_sub<R, NC, true>(u, vr[dir], vi[dir], ar, ai);
            }
#pragma unroll
            for (int a = 0; a < NC; ++a) {
                st_rows<S, NC>(Q, site, logW, j, a, ar[a], ai[a]);
                if (cg) {
                    R qr = ar[a], qi = ai[a];
                    St<S>::round(qr, qi);  // the dot products of the stored q
                    pqs = fmaR(vor[h][a], qr, fmaR(voi[h][a], qi, pqs));
                    qqs = fmaR(qr, qr, fmaR(qi, qi, qqs));
                    if (kDirect) {
                        rqs = fmaR(rr_[a], qr, fmaR(ri_[a], qi, rqs));
                        rps = fmaR(rr_[a], vor[h][a], fmaR(ri_[a], voi[h][a], rps));
                    }
                }
            }
        }
        acc[0] += (double)pqs;
        acc[1] += (double)rqs;
        acc[2] += (double)qqs;
        acc[3] += (double)rps;
    }
    if (!cg) return;
    if (kReuse) __syncthreads();  // every wavefront is done with the link tile
    block_partials<4>(bk, acc, W, logW, rd, sm);
}

struct HopB {  // kStHopB: where b comes from
    const double2 *b64;
    ProbeGen g;
    int gen;
};

// MODE 5 (W = 1): one right-hand side leaves a launch with one thread per
// site too few threads to fill the GPU (an 8^4 lattice: 16 workgroups), so
// a site takes 32 threads: thread (h, a) = (lane / 4, lane % 4) forms row a
// of hop h's product U v (rows a >= nc idle), the eight hops of a row are
// summed by a butterfly over lanes 4, 8 and 16 apart, and hop 0's threads
// write q.  Eight sites per workgroup pass.
template <typename S, typename LS, int NC, bool LINKS, int KIND>
__device__ __forceinline__ void k_stencil_split_body(const Blk &bk, Launch L, typename St<S>::R diag, const S *pin,
                                                     const S *__restrict__ rin, S *q, S *q2, const LS *__restrict__ U,
                                                     const int *__restrict__ nbr, int cg, Red rd, const HopB &hb) {
    constexpr bool HOP = KIND == kStHop || KIND == kStHopB;
    constexpr bool HOPB = KIND == kStHopB;
    constexpr bool INIT = KIND == kStInit;
    using R = typename St<S>::R;
    __shared__ double sm[4 * kBlock];
    const int tid = threadIdx.x, lane = tid & 31, h = lane >> 2, a = lane & 3;
    const int ngroups = (L.ns + 7) / 8;
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    for (int g = bk.b; g < ngroups; g += bk.nb) {
        const int item = g * 8 + (tid >> 5), site = item + (HOP ? L.ns : 0);
        const bool live = item < L.ns;
        R sr = 0, si = 0;
        if (live && a < NC) {
            const int y = nbr[site * 8 + h];
            if (LINKS) {
                // row a of U_mu(x) (h < 4) or of U_mu(x - mu)^H (h >= 4)
                const LS *u = U + ((size_t)site * 8 + h) * NC * NC;
#pragma unroll
                for (int b = 0; b < NC; ++b) {
                    typename St<LS>::R ur, ui;
                    St<LS>::ld(u, h < 4 ? a * NC + b : b * NC + a, ur, ui);
                    if (h >= 4) ui = -ui;
                    R vr, vi;
                    St<S>::ld(pin, (size_t)y * NC + b, vr, vi);
                    sr = fmaR((R)ur, vr, fmaR(-(R)ui, vi, sr));
                    si = fmaR((R)ur, vi, fmaR((R)ui, vr, si));
                }
            } else {
                St<S>::ld(pin, (size_t)y * NC + a, sr, si);
            }
        }
#pragma unroll
        for (int off = 4; off < 32; off <<= 1) {
            sr += __shfl_xor(sr, off, 64);
            si += __shfl_xor(si, off, 64);
        }
        if (live && h == 0 && a < NC) {
            if constexpr (HOPB) {
                double br = 0.0, bi = 0.0;
                if (!hb.gen)
                    St<double2>::ld(hb.b64, (size_t)site * NC + a, br, bi);
                else if (0 < hb.g.nvalid)
                    probe_value(hb.g, mix64(hb.g.seed), L.lat, NC, hb.g.rhs0, lex_of(L.lat, site), a, br, bi);
                sr += br;
                si += bi;
            }
            if (HOP) {
                St<S>::st(q, (size_t)site * NC + a, diag * sr, diag * si);
                continue;
            }
            R pr, pi;
            St<S>::ld(pin, (size_t)site * NC + a, pr, pi);
            R qr = fmaR(diag, pr, -sr), qi = fmaR(diag, pi, -si);
            St<S>::st(q, (size_t)site * NC + a, qr, qi);
            if (INIT) St<S>::st(q2, (size_t)site * NC + a, qr, qi);
            if (cg) {
                if (!INIT) acc[0] += (double)fmaR(pr, qr, pi * qi);
                acc[2] += (double)fmaR(qr, qr, qi * qi);
            }
        }
    }
    if (HOP || !cg) return;
    block_partials<4>(bk, acc, 1, 0, rd, sm);
}

template <typename S, typename LS, int NC, bool LINKS, int MODE, int KIND>
__global__ __launch_bounds__(kBlock) void k_stencil(Launch L, typename St<S>::R diag, const S *pin,
                                                    const S *__restrict__ rin, S *q, S *q2, const LS *__restrict__ U,
                                                    const int *__restrict__ nbr, int cg, Red rd, HopB hb) {
    // the bodies are inlined once with cg = 1 and once with cg = 0: with a
    // run-time flag the compiler keeps the registers of both paths live
    // (the BF16 body went from 69 to 187 registers)
    auto body = [&](int cg_) {
        if constexpr (MODE == 3 || MODE == 4)
            k_stencil_group_body<S, LS, NC, LINKS, MODE == 3 ? 2 : 4>(own_blk(), L, diag, pin, rin, q, U, nbr, cg_,
                                                                      rd);
        else if constexpr (MODE == 6)
            k_stencil_group_body<S, LS, NC, LINKS, 4, true>(own_blk(), L, diag, pin, rin, q, U, nbr, cg_, rd);
        else if constexpr (MODE == 5)
            k_stencil_split_body<S, LS, NC, LINKS, KIND>(own_blk(), L, diag, pin, rin, q, q2, U, nbr, cg_, rd, hb);
        else
            k_stencil_body<S, LS, NC, LINKS, MODE, KIND>(own_blk(), L, diag, pin, rin, q, q2, U, nbr, cg_, rd);
    };
    if constexpr (KIND == kStHop || KIND == kStHopB) {
        body(0);
    } else if constexpr (KIND == kStInit) {
        body(1);
    } else {
        if (cg)
            body(1);
        else
            body(0);
    }
}

// The vector update of a CG iteration (second kernel; alpha and beta from
// the finishing kernel): x += alpha p, r -= alpha q, p = r + beta p, and
// |r|^2 and Re q^H p of the new residual and direction as stored (the next
// finishing kernel adds the partials up).  A held or stopped lane keeps its
// direction (alpha = 0: x and r are unchanged too).
// The solution's update x += alpha p can be taken two iterations at a time
// (XM; FP32 or BF16 storage): an update with XM = 1 leaves x and records
// c = alpha_k / beta_k per lane; the next one (XM = 2) recovers the direction
// p_k it skipped from the two vectors it reads anyway, p_k = (p_{k+1} -
// r_{k+1}) / beta_k (the relation by which the skipped update formed p_{k+1}),
// and adds alpha_k p_k + alpha_{k+1} p_{k+1} in one read and write of x: six
// vector passes per iteration on average instead of seven.  The recovery
// divides by beta_k; its rounding error relative to alpha_k p_k is about
// eps / sqrt(beta_k) (|r_{k+1}| = sqrt(beta_k) |r_k| <= sqrt(beta_k) |p_k|),
// so a lane whose beta_k is below kDeferBetaMin (a restart has beta = 0)
// updates its x at once instead.  With BF16 storage the rounding of the
// stored p_{k+1} (2^-9 of it) enters the same way, about 2^-9 (1 + 1 /
// sqrt(beta_k)) of the step, against 2^-9 of the whole accumulated x that
// every BF16 write of x costs (and the pairs halve those writes); there the
// floor is 1/16 (at most 5 x 2^-9 of a step).  XM = 0 is the plain update.
// FP64 storage, whose result is x as it stands, takes the plain update alone:
// in pairs a step is rounded by up to 8 units of 2^-53 where it was by one
// (8^4 x 3 trace, W = 256, 2.31 ms for 2.40, but errors at 1e-15 of 1.05 times
// the plain ones' rms on the average of seven lattices and of 1.3 times on a
// 6^4 free field).
// An XM = 1 update is always followed by an XM = 2 one before anything
// reads x.
template <typename S>
constexpr double kDeferBetaMin = std::is_same<S, bf16x2>::value ? 1.0 / 16 : 1.0 / 64;

// XNT: x passes by the caches.  Of the vectors of an iteration x alone has no
// reader before the next update; where they are together larger than the
// 256 MB Infinity Cache (update_streams), keeping x out of it leaves the
// others more room.  16^4 x 3, FP32, W = 64 (290 MB): the fine trace 182 ms
// with x cached, 173 past the caches; where everything fits it only costs
// (8^4 x 3, FP64, W = 256, 140 MB: 2.44 ms and 2.54).
// XNT = 2: r and q too, from twice that size on, where little of them would
// last until its next reader (32^4 x 3, FP32, W = 32, 2.3 GB: 216.2 ms -> 214.2;
// 64 uneven lattices, BF16, over 1 GB: 57.0 -> 56.1; at 290 MB it costs, 16^4
// multi-shift, BF16, W = 128: 15.6 -> 16.0).
template <typename S, int XM, int XNT>
__device__ __forceinline__ void k_update_body(const Blk &bk, Launch L, S *__restrict__ x, S *__restrict__ r,
                                              S *__restrict__ p, const S *__restrict__ q, Red rd, CgState cs) {
    using R = typename St<S>::R;
    __shared__ double sm[2 * kBlock];
    const int tid = threadIdx.x, logW = L.logW, W = L.W;
    const int j = tid & (W - 1);
    const int sites_per_tile = kBlock >> logW;
    const R alpha = (R)ldg(cs.alpha + j);
    const double beta64 = ldg(cs.beta + j);
    const R beta = (R)beta64;
    const bool keep = (ldg(cs.flags + j) & kFlagHold) || !ldg(cs.active + j);
    // XM = 1: does this lane defer its x update (else it updates x now)?
    // XM = 2: the deferred coefficient alpha_k / beta_k (0: nothing deferred)
    const bool dfr = XM == 1 && !keep && beta64 >= kDeferBetaMin<S>;
    const bool xio = XM != 1 || (!keep && !dfr);
    const R cdef = XM == 2 ? (R)ldg(cs.xdef + j) : (R)0;
    if (XM == 1 && bk.b == 0 && tid < W) cs.xdef[j] = dfr ? ldg(cs.alpha + j) / beta64 : 0.0;
    double acc[2] = {0.0, 0.0};
    int t0, t1;
    tile_range(bk, L.ntiles, t0, t1);
    // element e = ((site * nc + a) << logW) + j: lane j is tid & (W-1) for
    // every e = e0 + tid + k * kBlock since kBlock is a multiple of W
    const size_t e0 = (size_t)t0 * sites_per_tile * L.nc * W;
    const size_t e1 = min((size_t)t1 * sites_per_tile, (size_t)L.ns) * L.nc * W;
    R part = 0, partq = 0;
    int cnt = 0;
    size_t e = e0 + tid;
    // four elements per pass, all loads issued before the first use (more
    // loads in flight per wavefront); the same summation order as the
    // element-by-element tail below; no branch inside (a kept direction is
    // stored back unchanged: a loaded value is stored exactly)
    for (; e + 3 * kBlock < e1; e += 4 * kBlock) {
        R xr[4], xi[4], rr_[4], ri[4], pr[4], pi[4], qr[4], qi[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            St<S>::ld(p, e + u * kBlock, pr[u], pi[u]);
            St<S>::template ld<(XNT > 1)>(q, e + u * kBlock, qr[u], qi[u]);
            St<S>::template ld<(XNT > 1)>(r, e + u * kBlock, rr_[u], ri[u]);
            if (xio) St<S>::template ld<(XNT > 0)>(x, e + u * kBlock, xr[u], xi[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            if (XM == 2) {
                xr[u] = fmaR(cdef, pr[u] - rr_[u], xr[u]);
                xi[u] = fmaR(cdef, pi[u] - ri[u], xi[u]);
            }
            if (xio)
                St<S>::template st<(XNT > 0)>(x, e + u * kBlock, fmaR(alpha, pr[u], xr[u]), fmaR(alpha, pi[u], xi[u]));
            rr_[u] = fmaR(-alpha, qr[u], rr_[u]);
            ri[u] = fmaR(-alpha, qi[u], ri[u]);
            St<S>::template st<(XNT > 1)>(r, e + u * kBlock, rr_[u], ri[u]);
            // the next iteration uses the stored (rounded) residual
            St<S>::round(rr_[u], ri[u]);
            R npr = keep ? pr[u] : fmaR(beta, pr[u], rr_[u]), npi = keep ? pi[u] : fmaR(beta, pi[u], ri[u]);
            St<S>::st(p, e + u * kBlock, npr, npi);
            St<S>::round(npr, npi);
            part = fmaR(rr_[u], rr_[u], fmaR(ri[u], ri[u], part));
            partq = fmaR(qr[u], npr, fmaR(qi[u], npi, partq));
        }
        if ((cnt += 4) == 24) {
            acc[0] += (double)part;
            acc[1] += (double)partq;
            part = partq = 0;
            cnt = 0;
        }
    }
    for (; e < e1; e += kBlock) {
        R xr, xi, rr_, ri, pr, pi, qr, qi;
        St<S>::ld(p, e, pr, pi);
        St<S>::template ld<(XNT > 1)>(q, e, qr, qi);
        St<S>::template ld<(XNT > 1)>(r, e, rr_, ri);
        if (xio) St<S>::template ld<(XNT > 0)>(x, e, xr, xi);
        if (XM == 2) {
            xr = fmaR(cdef, pr - rr_, xr);
            xi = fmaR(cdef, pi - ri, xi);
        }
        if (xio) St<S>::template st<(XNT > 0)>(x, e, fmaR(alpha, pr, xr), fmaR(alpha, pi, xi));
        rr_ = fmaR(-alpha, qr, rr_);
        ri = fmaR(-alpha, qi, ri);
        St<S>::template st<(XNT > 1)>(r, e, rr_, ri);
        St<S>::round(rr_, ri);
        R npr = keep ? pr : fmaR(beta, pr, rr_), npi = keep ? pi : fmaR(beta, pi, ri);
        St<S>::st(p, e, npr, npi);
        St<S>::round(npr, npi);
        part = fmaR(rr_, rr_, fmaR(ri, ri, part));
        partq = fmaR(qr, npr, fmaR(qi, npi, partq));
        if (++cnt == 24) {
            acc[0] += (double)part;
            acc[1] += (double)partq;
            part = partq = 0;
            cnt = 0;
        }
    }
    acc[0] += (double)part;
    acc[1] += (double)partq;
    // a kept direction keeps the Re q_prev^H p of the update that formed it
    // (the q loaded here is A of the kept direction itself): its total comes
    // back from cs.qp, once per lane
    if (keep) acc[1] = (bk.b == 0 && tid < W) ? ldg(cs.qp + j) : 0.0;
    block_partials_to<2>(bk, acc, W, logW, rd.part2, rd.nblk, sm);
}

template <typename S, int XM, int XNT>
__global__ __launch_bounds__(kBlock) void k_update(Launch L, S *__restrict__ x, S *__restrict__ r,
                                                   S *__restrict__ p, const S *__restrict__ q, Red rd, CgState cs) {
    k_update_body<S, XM, XNT>(own_blk(), L, x, r, p, q, rd, cs);
}

// Mixed precision: x64 += xlo, xlo = 0 (the low-precision iterate folded
// into the FP64 solution before a reliable update).  The first fold of a block
// sets x64 = xlo: the initialisation leaves x64 unwritten.
template <typename S>
__device__ __forceinline__ void k_fold_body(const Blk &bk, Launch L, double2 *__restrict__ x64, S *__restrict__ xlo,
                                            int first) {
    using R = typename St<S>::R;
    const int tid = threadIdx.x, W = L.W;
    const int sites_per_tile = kBlock >> L.logW;
    int t0, t1;
    tile_range(bk, L.ntiles, t0, t1);
    const size_t e0 = (size_t)t0 * sites_per_tile * L.nc * W;
    const size_t e1 = min((size_t)t1 * sites_per_tile, (size_t)L.ns) * L.nc * W;
    for (size_t e = e0 + tid; e < e1; e += kBlock) {
        R xr, xi;
        St<S>::ld(xlo, e, xr, xi);
        double2 v = first ? make_double2(0.0, 0.0) : x64[e];
        v.x += (double)xr;
        v.y += (double)xi;
        St<S>::st(xlo, e, 0, 0);
        x64[e] = v;
    }
}

template <typename S>
__global__ __launch_bounds__(kBlock) void k_fold(Launch L, double2 *__restrict__ x64, S *__restrict__ xlo,
                                                 int first) {
    k_fold_body<S>(own_blk(), L, x64, xlo, first);
}

// FP64 true residual r_new = b - A x64 with the FP64 hop links, |r_new|^2 per
// lane into rd.part2.  ru (a reliable update): r_new replaces the residual in the
// storage precision; a lane flagged to restart takes r_new as its direction.
// The other directions: FP32 storage continues them as p + (r_new - r_old),
// the direction the last update would have formed from r_new (so that
// r = p - beta p_prev still holds exactly for the finishing kernel), and
// sums Re q^H p of it (q = A p_prev, still in qin) beside |r_new|^2; BF16
// storage keeps them (residual replacement; its finishing kernel takes the
// exact line search along p) and writes the lane's total cs.qp back.
// Otherwise (statistics) nothing is written but the norm.
// ODD (even-odd order): the same walk over the odd sites, whose residual is made
// zero instead: xo = (b + H x64) / c (diag: 1 / c).  The FP64 stencil body that
// first did this holds all eight neighbours' values at once, 108 registers and
// two waves per SIMD (64 uneven lattices, BF16, W = 32: 308 us, 235 here; 16^4,
// FP32, W = 64: 107 and 104).
template <typename S, int NC, bool LINKS, int MODE, bool ODD = false>
__device__ __forceinline__ void k_true_resid_body(const Blk &bk, Launch L, double diag, const double2 *__restrict__ b64,
                                                  const double2 *__restrict__ x64, const double2 *__restrict__ U,
                                                  const int *__restrict__ nbr, S *__restrict__ rout,
                                                  S *__restrict__ pio, const S *__restrict__ qin, int ru, Red rd,
                                                  CgState cs, ProbeGen g, int gen, double2 *xo = nullptr) {
    constexpr int kMaxSites = kBlock / 16;
    // STAGE: two tile buffers, each the tile's hop links then its neighbour
    // indices; the next tile is copied into one while the other is read
    constexpr bool STAGE = MODE == 1 && LINKS;
    constexpr int kBufB = kMaxSites * 8 * NC * NC * 16 + kMaxSites * 8 * 4;
    __shared__ __align__(16) char sbuf[STAGE ? 2 * kBufB : 16];
    __shared__ int snb[MODE == 1 && !STAGE ? kMaxSites * 8 : 1];
    // the reduction at the end reuses the tile buffers when there are any
    __shared__ double sm_own[STAGE ? 1 : 2 * kBlock];
    double *sm = STAGE ? (double *)sbuf : sm_own;
    const int tid = threadIdx.x, logW = L.logW, W = L.W;
    const int j = tid & (W - 1);
    const int sl = MODE == 2 ? __builtin_amdgcn_readfirstlane(tid >> logW) : tid >> logW;
    const int sites_per_tile = kBlock >> logW;
    double acc[2] = {0.0, 0.0};
    const SiteWalk wk = site_walk(L, bk, ODD ? 1 : 0);
    const unsigned long long seedmix = gen ? mix64(g.seed) : 0ull;
    const ProbeLane pl = gen ? probe_lane(g, NC, g.rhs0 + j) : ProbeLane{};
    const bool restart = !ODD && ru && ((cs.flags[j] & kFlagRestart) || cs.ru_restart);
    if (STAGE && wk.first * sites_per_tile < wk.items)
        dma_tile<double2, NC>(sbuf, wk, wk.first * sites_per_tile, sites_per_tile, U, nbr);
    int cur = 0;
    for (int t = wk.first; t * sites_per_tile < wk.items; t += wk.stride, cur ^= 1) {
        const double *tsu = (const double *)(sbuf + cur * kBufB);  // this tile's hop links
        const int *tnb = (const int *)(sbuf + cur * kBufB + sites_per_tile * 8 * NC * NC * 16);
        if (STAGE) {
            // this tile's copy is complete, and every wavefront is done with the other buffer
            dma_wait_barrier();
            const int next0 = (t + wk.stride) * sites_per_tile;
            if (next0 < wk.items) dma_tile<double2, NC>(sbuf + (cur ^ 1) * kBufB, wk, next0, sites_per_tile, U, nbr);
        } else if (MODE == 1) {
            stage_nbr(snb, wk, t * sites_per_tile, sites_per_tile, nbr);
        }
        if (t * sites_per_tile + sl >= wk.items) continue;
        const int site = walk_site(wk, t * sites_per_tile + sl);
        int y[9];
        y[0] = site;
#pragma unroll
        for (int dir = 0; dir < 8; ++dir)
            y[dir + 1] = STAGE ? tnb[sl * 8 + dir] : (MODE == 1 ? snb[sl * 8 + dir] : ldg(nbr + site * 8 + dir));
        // Two halves: the site and its forward neighbours, then the backward
        // ones, each half's loads in flight together before its arithmetic
        // (all nine at once hold 108 registers of FP64 values: two waves per
        // SIMD instead of four)
        double vr[5][NC], vi[5][NC], br[NC], bi[NC];
#pragma unroll
        for (int k = ODD ? 1 : 0; k < 5; ++k) ld_site<double2, NC>(x64, y[k], logW, j, vr[k], vi[k]);
        if (gen) {
            // probes are regenerated instead of read back (exact values)
            const int x = lex_of(L.lat, site);
#pragma unroll
            for (int a = 0; a < NC; ++a) {
                br[a] = bi[a] = 0.0;
                if (j < g.nvalid) probe_at(g, seedmix, L.lat, NC, pl, x, a, br[a], bi[a]);
            }
        } else {
            ld_site<double2, NC>(b64, site, logW, j, br, bi);
        }
        // r = b - diag x + sum of hops: accumulated with the sign flipped
        double ar[NC], ai[NC];
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            ar[a] = ODD ? -br[a] : -fma(-diag, vr[0][a], br[a]);
            ai[a] = ODD ? -bi[a] : -fma(-diag, vi[0][a], bi[a]);
        }
#pragma unroll
        for (int dir = 0; dir < 8; ++dir) {
            if (dir == 4) {
                // the backward half: its loads wait until the forward values are spent
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 1; k < 5; ++k) ld_site<double2, NC>(x64, y[k + 4], logW, j, vr[k], vi[k]);
            }
            const int k = (dir & 3) + 1;
            if (!LINKS) {
#pragma unroll
                for (int a = 0; a < NC; ++a) {
                    ar[a] -= vr[k][a];
                    ai[a] -= vi[k][a];
                }
                continue;
            }
            double u[2 * NC * NC];
            if (STAGE) {
#pragma unroll
                for (int e = 0; e < 2 * NC * NC; ++e) u[e] = tsu[(sl * 8 + dir) * NC * NC * 2 + e];
            } else {
                ld_hop<double2, double, NC>(U, site, dir, u);
            }
            if (dir < 4)
                mul_sub<double, NC, false>(u, vr[k], vi[k], ar, ai);
            else
                mul_sub<double, NC, true>(u, vr[k], vi[k], ar, ai);
        }
        if constexpr (ODD) {
            double2 *xrow = xo + ((size_t)(site * NC) << logW);
#pragma unroll
            for (int a = 0; a < NC; ++a)
                St<double2>::st(xrow, ((size_t)a << logW) + j, -diag * ar[a], -diag * ai[a]);
            continue;
        }
        if (ru) {
            using R = typename St<S>::R;
            // (the neighbours' registers are free from here on)
            __builtin_amdgcn_sched_barrier(0);
            S *rrow = rout + ((size_t)(site * NC) << logW);
            S *prow = pio + ((size_t)(site * NC) << logW);
            const S *qrow = qin + ((size_t)(site * NC) << logW);
#pragma unroll
            for (int a = 0; a < NC; ++a) {
                const size_t i = ((size_t)a << logW) + j;
                R nr = (R)(-ar[a]), ni = (R)(-ai[a]);
                if (cs.rq_direct) {
                    St<S>::st(rrow, i, nr, ni);
                    if (restart) St<S>::st(prow, i, nr, ni);
                } else {
                    R ro_r, ro_i, po_r, po_i, qr, qi;
                    St<S>::ld(rrow, i, ro_r, ro_i);
                    St<S>::ld(prow, i, po_r, po_i);
                    St<S>::ld(qrow, i, qr, qi);
                    St<S>::st(rrow, i, nr, ni);
                    St<S>::round(nr, ni);
                    R npr = restart ? nr : po_r + (nr - ro_r), npi = restart ? ni : po_i + (ni - ro_i);
                    St<S>::st(prow, i, npr, npi);
                    St<S>::round(npr, npi);
                    acc[1] += (double)(qr * npr + qi * npi);
                }
            }
        }
#pragma unroll
        for (int a = 0; a < NC; ++a) acc[0] += ar[a] * ar[a] + ai[a] * ai[a];
    }
    if constexpr (ODD) return;
    if (ru && cs.rq_direct) acc[1] = (bk.b == 0 && tid < W) ? cs.qp[j] : 0.0;
    if (STAGE) __syncthreads();  // every wavefront is done with the tile buffers
    block_partials_to<2>(bk, acc, W, logW, rd.part2, rd.nblk, sm);
}

template <typename S, int NC, bool LINKS, int MODE>
__global__ __launch_bounds__(kBlock) void k_true_resid(Launch L, double diag, const double2 *__restrict__ b64,
                                                       const double2 *__restrict__ x64, const double2 *__restrict__ U,
                                                       const int *__restrict__ nbr, S *__restrict__ rout,
                                                       S *__restrict__ pio, const S *__restrict__ qin, int ru, Red rd,
                                                       CgState cs, ProbeGen g, int gen) {
    k_true_resid_body<S, NC, LINKS, MODE>(own_blk(), L, diag, b64, x64, U, nbr, rout, pio, qin, ru, rd, cs, g, gen);
}

template <int NC, bool LINKS, int MODE>
__global__ __launch_bounds__(kBlock) void k_odd_x(Launch L, double hop_scale, const double2 *__restrict__ b64,
                                                  double2 *x64, const double2 *__restrict__ U,
                                                  const int *__restrict__ nbr, ProbeGen g, int gen) {
    k_true_resid_body<double2, NC, LINKS, MODE, true>(own_blk(), L, hop_scale, b64, x64, U, nbr, nullptr, nullptr,
                                                      nullptr, 0, Red{}, CgState{}, g, gen, x64);
}

// The true residual from q64 = A x64 (the FP64 stencil, run just before on
// x64 with the FP64 hop links): r = b - q64 in FP64 element by element, with
// |r|^2 summed; with ru the inner-precision residual and direction are
// replaced as in k_true_resid_body (the FP32 continuation p += r_new - r,
// or p = r_new for a restarting lane) and Re q^H p of the new p summed.
// b is read, or regenerated from the probes (gen).
template <typename S, int NC>
__device__ __forceinline__ void k_resid_q_body(const Blk &bk, Launch L, const double2 *__restrict__ b64,
                                               const double2 *__restrict__ q64, S *__restrict__ rout,
                                               S *__restrict__ pio, const S *__restrict__ qin, int ru, Red rd,
                                               CgState cs, ProbeGen g, int gen) {
    using R = typename St<S>::R;
    __shared__ double sm[2 * kBlock];
    const int tid = threadIdx.x, logW = L.logW, W = L.W;
    const int j = tid & (W - 1);
    const int sites_per_tile = kBlock >> logW;
    const unsigned long long seedmix = gen ? mix64(g.seed) : 0ull;
    const ProbeLane pl = gen ? probe_lane(g, NC, g.rhs0 + j) : ProbeLane{};
    const bool restart = ru && ((ldg(cs.flags + j) & kFlagRestart) || cs.ru_restart);
    double acc[2] = {0.0, 0.0};
    int t0, t1;
    tile_range(bk, L.ntiles, t0, t1);
    // element e = ((site * NC + a) << logW) + j: lane j is tid % W for every
    // e = e0 + tid + k kBlock (kBlock is a multiple of W)
    const size_t e0 = (size_t)t0 * sites_per_tile * NC * W;
    const size_t e1 = min((size_t)t1 * sites_per_tile, (size_t)L.ns) * NC * W;
    for (size_t e = e0 + tid; e < e1; e += kBlock) {
        double qr, qi, br, bi;
        St<double2>::ld(q64, e, qr, qi);
        if (gen) {
            const int row = (int)(e >> logW), site = row / NC, a = row - site * NC;
            br = bi = 0.0;
            if (j < g.nvalid) probe_at(g, seedmix, L.lat, NC, pl, lex_of(L.lat, site), a, br, bi);
        } else {
            St<double2>::ld(b64, e, br, bi);
        }
        const double nr64 = br - qr, ni64 = bi - qi;
        acc[0] += nr64 * nr64 + ni64 * ni64;
        if (ru) {
            R nr = (R)nr64, ni = (R)ni64;
            if (cs.rq_direct) {
                St<S>::st(rout, e, nr, ni);
                if (restart) St<S>::st(pio, e, nr, ni);
            } else {
                R ro_r, ro_i, po_r, po_i, sqr, sqi;
                St<S>::ld(rout, e, ro_r, ro_i);
                St<S>::ld(pio, e, po_r, po_i);
                St<S>::ld(qin, e, sqr, sqi);
                St<S>::st(rout, e, nr, ni);
                St<S>::round(nr, ni);
                R npr = restart ? nr : po_r + (nr - ro_r), npi = restart ? ni : po_i + (ni - ro_i);
                St<S>::st(pio, e, npr, npi);
                St<S>::round(npr, npi);
                acc[1] += (double)(sqr * npr + sqi * npi);
            }
        }
    }
    if (ru && cs.rq_direct) acc[1] = (bk.b == 0 && tid < W) ? ldg(cs.qp + j) : 0.0;
    block_partials_to<2>(bk, acc, W, logW, rd.part2, rd.nblk, sm);
}

template <typename S, int NC>
__global__ __launch_bounds__(kBlock) void k_resid_q(Launch L, const double2 *__restrict__ b64,
                                                    const double2 *__restrict__ q64, S *__restrict__ rout,
                                                    S *__restrict__ pio, const S *__restrict__ qin, int ru, Red rd,
                                                    CgState cs, ProbeGen g, int gen) {
    k_resid_q_body<S, NC>(own_blk(), L, b64, q64, rout, pio, qin, ru, rd, cs, g, gen);
}

// t_j = sum_x sum_b conj(v_j(x,b)) x_j(x + p e0, b), probes regenerated.
__device__ __forceinline__ void k_displaced_dot_body(const Blk &bk, Launch L, ProbeGen g, int p,
                                                         const double2 *__restrict__ x64, Red rd, CgState cs) {
    __shared__ double sm[2 * kBlock];
    const int tid = threadIdx.x, logW = L.logW, W = L.W;
    const int j = tid & (W - 1), sl = tid >> logW;
    const int sites_per_tile = kBlock >> logW, nc = L.nc;
    const unsigned long long seedmix = mix64(g.seed);
    double acc[2] = {0.0, 0.0};
    int t0, t1;
    tile_range(bk, full_tiles(L), t0, t1);
    if (j < g.nvalid) {
        ProbeLane pl = probe_lane(g, nc, g.rhs0 + j);
        if (g.cmap) pl.c = g.cmap[pl.c];  // the parent class's probe: same noise, coarse colour
        for (int t = t0; t < t1; ++t) {
            const int site = t * sites_per_tile + sl;
            if (site >= L.lat.N || g.colors[site] != pl.c) continue;
            const int y = site_of(L.lat, shift0(L.lat, site, p));
            for (int b = 0; b < nc; ++b) {
                double zr, zi;
                probe_at(g, seedmix, L.lat, nc, pl, site, b, zr, zi);
                if (zr == 0.0 && zi == 0.0) continue;
                const double2 xv = x64[((size_t)(y * nc + b) << logW) + j];
                acc[0] += zr * xv.x + zi * xv.y;  // conj(z) * x
                acc[1] += zr * xv.y - zi * xv.x;
            }
        }
    }
    block_partials<2>(bk, acc, W, logW, rd, sm);
}

// Map of a nested colouring's fine colours to coarse ones (three passes:
// clear, scatter, check; every colour is range-checked before it indexes).
__global__ void k_level_map_clear(int *cmap, int nfine, int *bad) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nfine) cmap[i] = -1;
    if (i == 0) *bad = 0;
}

__global__ void k_level_map_scatter(int N, const int *fine, int nfine, const int *coarse, int ncoarse, int *cmap,
                                    int *bad) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= N) return;
    const int c = fine[x], cc = coarse[x];
    if (c < 0 || c >= nfine || cc < 0 || cc >= ncoarse) {
        *bad = 1;
        return;
    }
    cmap[c] = cc;  // equal values from every site of a nested colouring
}

__global__ void k_level_map_check(int N, const int *fine, int nfine, const int *coarse, const int *cmap, int *bad) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= N) return;
    const int c = fine[x];
    if (c >= 0 && c < nfine && cmap[c] != coarse[x]) *bad = 1;
}

__global__ __launch_bounds__(kBlock) void k_displaced_dot(Launch L, ProbeGen g, int p,
                                                         const double2 *__restrict__ x64, Red rd, CgState cs) {
    k_displaced_dot_body(own_blk(), L, g, p, x64, rd, cs);
}

// t_j = a_j^H b_j (FP64 vectors)
__device__ __forceinline__ void k_dot_body(const Blk &bk, Launch L, const double2 *__restrict__ a64,
                                               const double2 *__restrict__ b64, Red rd, CgState cs) {
    __shared__ double sm[2 * kBlock];
    const int tid = threadIdx.x, W = L.W;
    const int sites_per_tile = kBlock >> L.logW;
    double acc[2] = {0.0, 0.0};
    int t0, t1;
    tile_range(bk, full_tiles(L), t0, t1);
    const size_t e0 = (size_t)t0 * sites_per_tile * L.nc * W;
    const size_t e1 = min((size_t)t1 * sites_per_tile, (size_t)L.lat.N) * L.nc * W;
    for (size_t e = e0 + tid; e < e1; e += kBlock) {
        const double2 u = a64[e], v = b64[e];
        acc[0] += u.x * v.x + u.y * v.y;
        acc[1] += u.x * v.y - u.y * v.x;
    }
    block_partials<2>(bk, acc, W, L.logW, rd, sm);
}

__global__ __launch_bounds__(kBlock) void k_dot(Launch L, const double2 *__restrict__ a64,
                                               const double2 *__restrict__ b64, Red rd, CgState cs) {
    k_dot_body(own_blk(), L, a64, b64, rd, cs);
}

// Adjoint force of one block of right-hand sides, one thread per output
// entry (site, mu, a, b):
//   dU[mu][x][a][b]    (+)= scale * sum_j conj(l_j(x)_a) x_j(x+mu)_b
//   dUbar[mu][x][a][b] (+)= scale * sum_j x_j(x)_a conj(l_j(x+mu)_b)
__global__ __launch_bounds__(kBlock) void k_force(Launch L, const double2 *__restrict__ x64,
                                                 const double2 *__restrict__ l64, const int *__restrict__ nbr,
                                                 double scale, int first, double2 *__restrict__ dU,
                                                 double2 *__restrict__ dUbar) {
    const int nc = L.nc, W = L.W, logW = L.logW;
    const long long n = (long long)L.lat.N * 4 * nc * nc;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int b = (int)(e % nc);
    const int a = (int)((e / nc) % nc);
    const int mu = (int)((e / (nc * nc)) % 4);
    const int site = (int)(e / (4 * nc * nc));
    const int y = nbr[site * 8 + mu];
    double ur = 0, ui = 0, vr = 0, vi = 0;
    const double2 *la = l64 + ((size_t)(site * nc + a) << logW);
    const double2 *xb = x64 + ((size_t)(y * nc + b) << logW);
    const double2 *xa = x64 + ((size_t)(site * nc + a) << logW);
    const double2 *lb = l64 + ((size_t)(y * nc + b) << logW);
    for (int j = 0; j < W; ++j) {
        const double2 l1 = la[j], x1 = xb[j], x2 = xa[j], l2 = lb[j];
        ur += l1.x * x1.x + l1.y * x1.y;  // conj(l) x
        ui += l1.x * x1.y - l1.y * x1.x;
        vr += x2.x * l2.x + x2.y * l2.y;  // x conj(l)
        vi += x2.y * l2.x - x2.x * l2.y;
    }
    const size_t o = ((size_t)mu * L.lat.N + lex_of(L.lat, site)) * nc * nc + a * nc + b;
    double2 du = make_double2(scale * ur, scale * ui), db = make_double2(scale * vr, scale * vi);
    if (!first) {
        if (dU) {
            const double2 t = dU[o];
            du.x += t.x;
            du.y += t.y;
        }
        if (dUbar) {
            const double2 t = dUbar[o];
            db.x += t.x;
            db.y += t.y;
        }
    }
    if (dU) dU[o] = du;
    if (dUbar) dUbar[o] = db;
}

// internal FP64 -> ABI [rhs][site][nc] for lanes < nvalid
__global__ void k_to_abi(Launch L, const double2 *__restrict__ x64, double2 *__restrict__ xabi, long long rhs0,
                         long long nvalid) {
    const long long n = (long long)L.lat.N * L.nc * L.W;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int j = (int)(e & (L.W - 1));
    if (j >= nvalid) return;
    const int sa = (int)(e >> L.logW), site = sa / L.nc, a = sa - site * L.nc;
    xabi[((size_t)(rhs0 + j) * L.lat.N + lex_of(L.lat, site)) * L.nc + a] = x64[e];
}

template <typename S>
__global__ void k_abi_to_internal(Launch L, const double2 *__restrict__ vabi, long long rhs0, long long nvalid,
                                  S *__restrict__ out) {
    const long long n = (long long)L.lat.N * L.nc * L.W;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int j = (int)(e & (L.W - 1));
    const long long sa = e >> L.logW;
    double re = 0, im = 0;
    if (j < nvalid) {
        const double2 v = vabi[(size_t)(rhs0 + j) * L.lat.N * L.nc + sa];
        re = v.x;
        im = v.y;
    }
    St<S>::st(out, e, (typename St<S>::R)re, (typename St<S>::R)im);
}

template <typename S>
__global__ void k_internal_to_abi(Launch L, const S *__restrict__ in, double2 *__restrict__ yabi, long long rhs0,
                                  long long nvalid) {
    const long long n = (long long)L.lat.N * L.nc * L.W;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int j = (int)(e & (L.W - 1));
    if (j >= nvalid) return;
    typename St<S>::R re, im;
    St<S>::ld(in, e, re, im);
    yabi[(size_t)(rhs0 + j) * L.lat.N * L.nc + (e >> L.logW)] = make_double2((double)re, (double)im);
}

// probes in the ABI layout [rhs][site][nc]
__global__ void k_probes_abi(Lat lat, int nc, ProbeGen g, long long nrhs, double2 *__restrict__ out) {
    const long long n = nrhs * lat.N * nc;
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const int b = (int)(e % nc);
    const int site = (int)((e / nc) % lat.N);
    const long long jj = e / ((long long)nc * lat.N);
    double re, im;
    probe_value(g, mix64(g.seed), lat, nc, g.rhs0 + jj, site, b, re, im);
    out[e] = make_double2(re, im);
}

// ============================================================ multi-instance launches
//
// One launch covers every slot (job) of a batch: workgroup w belongs to slot
// slot_of[w] and runs the same body as a standalone launch on that slot's
// lattice, with the slot's own buffers.  Slots whose flags do not include
// the kernel's phase return at once.  The descriptors live in device memory
// and are rewritten by the host between launches, so a captured graph of
// these launches stays valid while finished slots are refilled.

__device__ __forceinline__ const SlotDesc *slot_of_block(const BatchLaunch &B, Blk &bk, int phase) {
    const int s = B.slot_of[blockIdx.x];
    const SlotDesc *d = B.sd + s;
    if (!(d->flags & phase)) return nullptr;
    // an iterating slot whose lanes all stopped at a reliable update waits,
    // idle, for the host to retire it at its next check
    if (phase == kSlotIter && d->cs.live && ldg(d->cs.live) == 0) return nullptr;
    bk.b = (int)blockIdx.x - d->blk0;
    bk.nb = d->L.nblk;
    return d;
}

template <typename S>
__global__ __launch_bounds__(kBlock) void k_b_init(BatchLaunch B) {
    Blk bk;
    const SlotDesc *d = slot_of_block(B, bk, kSlotInit);
    if (!d) return;
    k_init_body<S, 0>(bk, d->L, d->g, nullptr, 0, 0, (double2 *)d->b64, (S *)d->r, (S *)d->p,
                      (S *)d->xlo, 1.0 / d->diag, d->rd);
}

// the same in even-odd order
template <typename S, int NC, bool LINKS>
__global__ __launch_bounds__(kBlock) void k_b_init_probe(BatchLaunch B) {
    Blk bk;
    const SlotDesc *d = slot_of_block(B, bk, kSlotInit);
    if (!d) return;
    k_init_probe_body<S, NC, LINKS>(bk, d->L, d->g, (S *)d->r, (S *)d->p, (S *)d->xlo, 1.0 / d->diag,
                                    (const double2 *)d->U64, d->rd);
}

// KIND kStFull: q = A p (even-odd: its even half); kStHop: the odd half of p.
template <typename S, typename LS, int NC, bool LINKS, int MODE, int KIND>
__global__ __launch_bounds__(kBlock) void k_b_stencil(BatchLaunch B) {
    Blk bk;
    const SlotDesc *d = slot_of_block(B, bk, kSlotIter);
    if (!d) return;
    if constexpr (KIND == kStHop)
        k_stencil_body<S, LS, NC, LINKS, MODE, KIND>(bk, d->L, (typename St<S>::R)(1.0 / d->diag), (const S *)d->p,
                                                     nullptr, (S *)d->p, nullptr, (const LS *)d->U, d->nbr, 0, d->rd);
    else
        k_stencil_body<S, LS, NC, LINKS, MODE, KIND>(bk, d->L, (typename St<S>::R)d->diag, (const S *)d->p,
                                                     (const S *)d->r, (S *)d->q, nullptr, (const LS *)d->U, d->nbr, 1,
                                                     d->rd);
}

// Even-odd order: the odd half of the FP64 solution, x_o = (b_o + H x_e) / c
template <int NC, bool LINKS, int MODE>
__global__ __launch_bounds__(kBlock) void k_b_odd_x(BatchLaunch B, int phase) {
    Blk bk;
    const SlotDesc *d = slot_of_block(B, bk, phase);
    if (!d) return;
    k_true_resid_body<double2, NC, LINKS, MODE, true>(bk, d->L, 1.0 / d->diag, (const double2 *)d->b64,
                                                      (const double2 *)d->x64, (const double2 *)d->U64, d->nbr, nullptr,
                                                      nullptr, nullptr, 0, d->rd, d->cs, d->g, d->gen_b,
                                                      (double2 *)d->x64);
}

template <typename S, int XM, int XNT>
__global__ __launch_bounds__(kBlock) void k_b_update(BatchLaunch B) {
    Blk bk;
    const SlotDesc *d = slot_of_block(B, bk, kSlotIter);
    if (!d) return;
    // FP64: the iterate is x64 itself (xlo aliases it)
    k_update_body<S, XM, XNT>(bk, d->L, (S *)d->xlo, (S *)d->r, (S *)d->p, (const S *)d->q,
                         d->rd, d->cs);
}

template <typename S>
__global__ __launch_bounds__(kBlock) void k_b_fold(BatchLaunch B, int phase) {
    Blk bk;
    const SlotDesc *d = slot_of_block(B, bk, phase);
    if (!d) return;
    k_fold_body<S>(bk, d->L, (double2 *)d->x64, (S *)d->xlo, d->fold0);
}

template <typename S, int NC, bool LINKS, int MODE>
__global__ __launch_bounds__(kBlock) void k_b_true_resid(BatchLaunch B, int phase, int ru) {
    Blk bk;
    const SlotDesc *d = slot_of_block(B, bk, phase);
    if (!d) return;
    k_true_resid_body<S, NC, LINKS, MODE>(bk, d->L, d->diag, (const double2 *)d->b64,
                                          (const double2 *)d->x64, (const double2 *)d->U64, d->nbr,
                                          (S *)d->r, (S *)d->p, (const S *)d->q, ru, d->rd,
                                          d->cs, d->g, d->gen_b);
}

__global__ __launch_bounds__(kBlock) void k_b_dot(BatchLaunch B) {
    Blk bk;
    const SlotDesc *d = slot_of_block(B, bk, kSlotFinal);
    if (!d) return;
    k_displaced_dot_body(bk, d->L, d->g, d->disp, (const double2 *)d->x64, d->rd, d->cs);
}

// one workgroup per (slot, lane)
template <int NV, int EPI>
__global__ __launch_bounds__(kBlock) void k_b_finish(BatchLaunch B, int phase) {
    const int s = blockIdx.x / B.W, lane = blockIdx.x % B.W;
    const SlotDesc *d = B.sd + s;
    if (!(d->flags & phase) || lane >= d->L.W) return;
    k_finish_body<NV, EPI>(lane, d->rd, d->cs);
}

// After the workgroups were shared anew among the slots, the |r|^2 and
// Re q^H p partials of an iterating slot (written by its last update with its
// old number of workgroups) are replaced by the lane's totals, cs.rr and
// cs.qp (which the check before the new sharing took from them): partial 0
// holds them, the others 0.
__global__ __launch_bounds__(kBlock) void k_b_reseed(BatchLaunch B) {
    const int s = blockIdx.x / B.W, lane = blockIdx.x % B.W;
    const SlotDesc *d = B.sd + s;
    if (!(d->flags & kSlotIter) || lane >= d->L.W) return;
    const double rr = d->cs.rr[lane], qp = d->cs.qp[lane];
    double *dst = d->rd.part2 + (size_t)lane * d->rd.nblk * 2;
    for (int b = threadIdx.x; b < d->rd.nblk; b += kBlock) {
        dst[2 * b] = b == 0 ? rr : 0.0;
        dst[2 * b + 1] = b == 0 ? qp : 0.0;
    }
}

// One wavefront per (slot, lane): wavefront g = blockIdx.x * 4 + wave takes
// slot g / W, lane g % W (a slot's few dozen partials per lane need no
// more; with a workgroup per lane the launch was mostly idle threads).
__global__ __launch_bounds__(kBlock) void k_b_finish_cg(BatchLaunch B) {
    const int g = blockIdx.x * (kBlock / 64) + (int)(threadIdx.x >> 6);
    const int s = g / B.W, lane = g % B.W;
    if (s >= B.nslots) return;
    const SlotDesc *d = B.sd + s;
    if (!(d->flags & kSlotIter) || lane >= d->L.W || (d->cs.live && ldg(d->cs.live) == 0)) return;
    k_finish_cg_wave_body(lane, d->rd, d->cs);
}

// One workgroup per (slot, lane).
__global__ __launch_bounds__(kBlock) void k_b_finish_cg_wide(BatchLaunch B) {
    const int s = blockIdx.x / B.W, lane = blockIdx.x % B.W;
    const SlotDesc *d = B.sd + s;
    if (!(d->flags & kSlotIter) || lane >= d->L.W || (d->cs.live && ldg(d->cs.live) == 0)) return;
    k_finish_cg_body(lane, d->rd, d->cs);
}

__global__ void k_b_ctrl(BatchLaunch B) {
    const SlotDesc *d = B.sd + blockIdx.x;
    k_ctrl_body(d->cs, d->L.W);
}

// ============================================================ small solves
//
// k_small: the whole CG solve of a block in one launch, for problems whose
// step is a few microseconds of work: with a launch per kernel a step of one
// 8^4 x 3 right-hand side took 30 us for 16 us of kernels that each mostly
// start, wait for memory and drain.  A group of workgroups (one per CU, all
// resident) solves WG right-hand sides, several groups the lanes of a block
// side by side, and the workgroups of a group meet at two sums per step:
//   A   p = r + beta p, p_o = H p / c on the odd sites, with |p|^2 and
//       |p_o|^2; p^H S p = c (|p|^2 - |p_o|^2), hence alpha
//   B   q = c p - H p_o on the even sites, r -= alpha q, x += alpha p, with
//       |r|^2, hence beta
// (index order: A forms q = A p on every site with p^H q, B updates).
//
// Eight threads share a site, one per hop.  A thread keeps, for the whole
// solve, the matrix of its hop into its odd and into its even site, and the
// direction p at the even neighbour its odd site's hop comes from, which it
// advances itself from r there: p is never stored.  The hop sums are
// reduce-scattered over the eight threads (seven exchanges), after which
// thread h holds real component h of the site and keeps that component of r,
// p and x.  A step loads the neighbours' r and p_o and stores one component of
// each, nothing else.
//
// After convergence x_o = (b_o + H x) / c and the true residual; with `refine`
// (mixed-precision requests, whose stopping rule is the true residual) lanes
// that miss the tolerance go on from it.
//
// Memory between workgroups.  Stores that others read go through agent-scope
// atomics, past the L2 of their XCD, and have completed (s_waitcnt) before the
// workgroup's partial sums are stored, which everyone waits for and which are
// their own flags: each half of a double travels in a word with the number of
// the sum (one more round trip for separate flags: 8.0 -> 7.5 us a step).
// The vectors are loaded as usual, through the caches, which is coherent
// because no address is loaded from a cache that may hold an older value:
// every step writes its r and p_o to a slot of a ring that nothing has read
// since the last agent-scope acquire (which drops the caches' lines: the start
// of every launch is one, and there is one whenever the ring wraps), a
// workgroup's share of a vector is whole 128-byte lines, and a slot is read
// only after the sum that follows its writing.  (An acquire in every sum took
// 9 us with 64 workgroups and 32 with 256: they queue at the XCD's L2.)
// Every wait is bounded: should some workgroup not become resident (other
// work holding the CUs), all give up, set *err and the host solves the block
// with the launched kernels instead; *stop keeps the launches already queued
// behind from waiting in their turn.

__device__ __forceinline__ double ldc(const double *p) {
    return __builtin_bit_cast(double, __hip_atomic_load((const unsigned long long *)p, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT));
}
__device__ __forceinline__ void stc(double *p, double v) {
    __hip_atomic_store((unsigned long long *)p, __builtin_bit_cast(unsigned long long, v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}

// v of the thread whose index differs in the bits of CTRL's permutation
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)u, CTRL, 0xf, 0xf, false);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(u >> 32), CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// Sum of the eight threads' t[h] over an aligned group of eight threads, in
// the thread with index h in the group.  Three halvings between threads i and
// i ^ 7, i ^ 3, i ^ 1 (lane permutations inside the vector unit): each keeps
// the half of its values that holds its own.
__device__ __forceinline__ double reduce_scatter8(const double (&t)[8], int h) {
    double u[4], w[2];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const double keep = (h & 4) ? t[k + 4] : t[k], give = (h & 4) ? t[k] : t[k + 4];
        u[k] = keep + dpp<0x141>(give);  // row_half_mirror: i ^ 7
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double keep = (h & 2) ? u[k + 2] : u[k], give = (h & 2) ? u[k] : u[k + 2];
        w[k] = keep + dpp<0x1B>(give);  // quad_perm 3, 2, 1, 0: i ^ 3
    }
    const double keep = (h & 1) ? w[1] : w[0], give = (h & 1) ? w[0] : w[1];
    return keep + dpp<0xB1>(give);  // quad_perm 1, 0, 3, 2: i ^ 1
}

struct SmallShared {
    double sm[kSmallThreads / 64][8];
    double out[4];
    int any;
};

// Sums over the workgroups of a group of the values v[k] (k < 2 WG), in a
// fixed order (threads, wavefronts, workgroups), and a barrier among them.
// Thread l < WG then calls step(v[2l], v[2l + 1]), the scalar part of lane l's
// iteration (in every workgroup, with the same values), which returns what
// every thread gets in out[l]; any: whether some lane's `active` is set after
// it.  False when a wait ran out.
template <int WG, typename F>
__device__ __forceinline__ bool small_sum(const SmallArgs &A, SmallShared &sh, int polls, unsigned &tag,
                                          const double (&v)[8], const int &active, F step, double (&out)[WG],
                                          int &any) {
    const int tid = threadIdx.x, n = A.nwg, lane = tid & 63, wave = tid >> 6;
    const int group = blockIdx.x % A.ngroups, wb = blockIdx.x / A.ngroups;
    auto wave_sum = [&](double a) {  // a: value tid % 8
        a += __shfl_xor(a, 8, 64);
        a += __shfl_xor(a, 16, 64);
        a += __shfl_xor(a, 32, 64);
        if (lane < 8) sh.sm[wave][lane] = a;
    };
    auto total = [&]() {
        double a = 0.0;
        if (tid < 8)
#pragma unroll
            for (int k = 0; k < kSmallThreads / 64; ++k) a += sh.sm[k][tid];
        return a;
    };
    ++tag;
    wave_sum(reduce_scatter8(v, tid & 7));
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wavefront's stores have completed
    __syncthreads();                     // and the workgroup's
    unsigned long long *part = A.part + ((size_t)(tag & 1) * A.ngroups + group) * n * 16;
    const unsigned long long mark = (unsigned long long)tag << 32;
    if (tid < 8) {
        const unsigned long long u = __builtin_bit_cast(unsigned long long, total());
        unsigned long long *e = part + ((size_t)wb * 8 + tid) * 2;
        __hip_atomic_store(e, mark | (u & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(e + 1, mark | (u >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    int good = 1;
    double a = 0.0;
    for (int w = tid >> 3; w < n; w += kSmallThreads >> 3) {  // (polls: of all its words together)
        const unsigned long long *e = part + ((size_t)w * 8 + (tid & 7)) * 2;
        unsigned long long lo = 0, hi = 0;
        for (; polls > 0; --polls) {
            lo = __hip_atomic_load(e, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            hi = __hip_atomic_load(e + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if ((lo >> 32) == tag && (hi >> 32) == tag) break;
        }
        good &= polls > 0;
        a += __builtin_bit_cast(double, (hi << 32) | (lo & 0xffffffffull));
    }
    if (!__syncthreads_and(good)) return false;
    wave_sum(a);
    __syncthreads();
    if (wave == 0) {
        a = total();
        const double t0 = __shfl(a, (2 * tid) & 63, 64), t1 = __shfl(a, (2 * tid + 1) & 63, 64);
        if (tid < WG) sh.out[tid] = step(t0, t1);
        const int some = __any(tid < WG && active);
        if (tid == 0) sh.any = some;
    }
    __syncthreads();
#pragma unroll
    for (int l = 0; l < WG; ++l) out[l] = sh.out[l];
    any = sh.any;
    return true;
}

__global__ __launch_bounds__(kBlock) void k_small_clear(unsigned long long *part) {
    stg(part + (size_t)blockIdx.x * kBlock + threadIdx.x, 0ull);
}

__global__ void k_small_go(unsigned *stop) { stg(stop, 0u); }

template <int NC, bool LINKS, bool EO, int WG>
__global__ __launch_bounds__(kSmallThreads) void k_small(SmallArgs A) {
    static_assert(2 * WG <= 8, "two sums per lane");
    __shared__ SmallShared sh;
    // with four lanes the matrices live in LDS ([element][thread], up to 144 KB
    // of a CU's 160), where with them in registers 176 spilled; with fewer in
    // registers (two lanes: 374 us a solve of 16 right-hand sides, 417 from LDS)
    constexpr bool kLds = LINKS && WG > 2;
    __shared__ double2 su[kLds ? (EO ? 2 : 1) * NC * NC * kSmallThreads : 1];
    const int tid = threadIdx.x, h = tid & 7;
    const int group = blockIdx.x % A.ngroups, wb = blockIdx.x / A.ngroups;
    const int ns = A.ns, s = wb * (kSmallThreads / 8) + (tid >> 3);
    const bool live = s < ns;
    // this thread's component of its sites: colour ca, real or imaginary part
    const bool own = live && h < 2 * NC;
    const int ca = own ? h >> 1 : 0, im = h & 1;
    // the launches queued behind one that gave up end at their first sum
    // (loaded here, waited for there)
    const int polls = __hip_atomic_load(A.stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 0 : A.polls;
    const double c = A.c, ic = 1.0 / A.c;
    const unsigned long long seedmix = A.src == 0 ? mix64(A.g.seed) : 0ull;
    const CgState &cs = A.cs;
    // the hops into site s (odd: site ns + s of the even-odd order): the
    // neighbour's index in its half, and the matrix (conjugate transposed for
    // a backward hop)
    struct Hop {
        int y;
        double2 u[LINKS && !kLds ? NC * NC : 1];
        double2 *lds;
    };
    auto load_hop = [&](int site, int half) {
        Hop g{};
        g.lds = su + (kLds ? half * NC * NC * kSmallThreads + tid : 0);
        if (live) g.y = ldg(A.nbr + (size_t)site * 8 + h);
        if (LINKS) {
            const double2 *u = (const double2 *)A.U + ((size_t)(live ? site : 0) * 8 + h) * NC * NC;
#pragma unroll
            for (int a = 0; a < NC; ++a)
#pragma unroll
                for (int b = 0; b < NC; ++b) {
                    double2 e = ldg(u + (h < 4 ? a * NC + b : b * NC + a));
                    if (h >= 4) e.y = -e.y;
                    if (kLds) g.lds[(a * NC + b) * kSmallThreads] = e;  // (read by this thread only)
                    else g.u[a * NC + b] = e;
                }
        }
        return g;
    };
    const Hop he = load_hop(s, 0), ho = EO ? load_hop(ns + s, 1) : he;
    const int ye = EO ? he.y - ns : he.y, yo = ho.y;  // (an even site's neighbours are odd)
    // component `own` of the sum over the hops of U v
    auto hop_sum = [&](const Hop &g, const double2 (&v)[NC]) {
        double t[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int a = 0; a < NC; ++a) {
            if (!LINKS) {
                t[2 * a] = v[a].x;
                t[2 * a + 1] = v[a].y;
                continue;
            }
#pragma unroll
            for (int b = 0; b < NC; ++b) {
                const double2 e = kLds ? g.lds[(a * NC + b) * kSmallThreads] : g.u[kLds ? 0 : a * NC + b];
                t[2 * a] = fma(e.x, v[b].x, fma(-e.y, v[b].y, t[2 * a]));
                t[2 * a + 1] = fma(e.x, v[b].y, fma(e.y, v[b].x, t[2 * a + 1]));
            }
        }
        return reduce_scatter8(t, h);
    };
    // vectors of the group's ring: element (site of a half, colour, lane l)
    double2 *ring = (double2 *)A.ring + (size_t)group * A.nring * 2 * A.vec;
    auto Rk = [&](int k) { return ring + (size_t)(2 * k) * A.vec; };
    auto Wk = [&](int k) { return ring + (size_t)(2 * k + 1) * A.vec; };
    auto publish = [&](double2 *v, int l, double x) {
        if (own) stc((double *)(v + ((size_t)(s * NC + ca) * WG + l)) + im, x);
    };
    auto gather = [&](const double2 *v, int y, int l, double2 (&out)[NC]) {
#pragma unroll
        for (int b = 0; b < NC; ++b)
            out[b] = live ? ldg(v + ((size_t)(y * NC + b) * WG + l)) : make_double2(0.0, 0.0);
    };

    unsigned tag = A.tag;
    int cur = 0;
    double v[8], out[WG];
    auto give_up = [&]() {
        if (tid != 0) return;
        __hip_atomic_store(A.stop, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *A.err = 1;
    };
    auto advance = [&]() {
        cur = cur + 1 < A.nring ? cur + 1 : 0;
        // the slots are read a second time from here on
        if (cur == 0) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    };
    // blocks of WG lanes, the group's share of the W lanes in turn
    for (int l0 = group * WG; l0 < A.W; l0 += A.ngroups * WG) {
        if (l0 >= A.nvalid) {  // lanes without a right-hand side: x = 0
            for (int j = l0; j < min(l0 + WG, A.W); ++j) {
                if (own) {
                    A.x[2 * ((size_t)(s * NC + ca) * A.W + j) + im] = 0.0;
                    if (EO) A.x[2 * ((size_t)((ns + s) * NC + ca) * A.W + j) + im] = 0.0;
                }
                if (wb != 0 || tid != 0) continue;
                cs.rr[j] = cs.qp[j] = cs.rr_ref[j] = cs.bb[j] = cs.alpha[j] = cs.beta[j] = cs.true_rr[j] = 0.0;
                cs.active[j] = cs.iters[j] = 0;
                cs.flags[j] = kFlagConverged;
            }
            continue;
        }
        // b at a site (of the internal order), colour a, lane l of this block
        auto b_at = [&](int site, int a, int l) {
            double re = 0.0, bi = 0.0;
            const int x = lex_of(A.lat, site), j = l0 + l;
            if (j < A.nvalid) {
                if (A.src == 0) {
                    const ProbeLane pl = probe_lane(A.g, NC, A.g.rhs0 + j);
                    probe_at(A.g, seedmix, A.lat, NC, pl, x, a, re, bi);
                } else {
                    const double2 t = ldg((const double2 *)A.b +
                                          (A.src == 1 ? ((size_t)(A.rhs0 + j) * A.lat.N + x) * NC + a
                                                      : (size_t)(x * NC + a) * A.W + j));
                    re = t.x;
                    bi = t.y;
                }
            }
            return make_double2(re, bi);
        };
        auto b_own = [&](int site, int l) {
            if (!own) return 0.0;
            const double2 t = b_at(site, ca, l);
            return im ? t.y : t.x;
        };
        // own components, and p at the neighbour of the A phase's hop
        double r[WG], p[WG], x[WG], q[WG];
        double2 pn[WG][NC];
        int it = 0, nref = 0, any;
        // the scalars of lane l, in thread l
        double rr = 0.0, bb = 0.0, rr_first = 0.0, true_rr = 0.0;
        int active = 0, flags = 0, iters = 0;
        const auto none = [](double, double) { return 0.0; };
        const auto clear = [&]() {
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = 0.0;
        };
        // the top of an iteration: a lane that meets the tolerance stops
        const auto check = [&]() {
            if (active && rr <= cs.tol2 * bb) {
                active = 0;
                flags |= kFlagConverged;
            }
        };

        // first residual, |r|^2 and |b|^2
        clear();
#pragma unroll
        for (int l = 0; l < WG; ++l) {
            r[l] = b_own(s, l);
            v[2 * l + 1] = r[l] * r[l];
            if (EO) {
                const double bo = b_own(ns + s, l);
                v[2 * l + 1] += bo * bo;
                double2 t[NC];
#pragma unroll
                for (int b = 0; b < NC; ++b) t[b] = live ? b_at(he.y, b, l) : make_double2(0.0, 0.0);
                const double g = hop_sum(he, t);
                if (own) r[l] = fma(ic, g, r[l]);
            }
            v[2 * l] = r[l] * r[l];
            p[l] = x[l] = 0.0;
#pragma unroll
            for (int b = 0; b < NC; ++b) pn[l][b] = make_double2(0.0, 0.0);
            publish(Rk(cur), l, r[l]);
        }
        double beta[WG];
        if (!small_sum<WG>(A, sh, polls, tag, v, active,
                           [&](double t0, double t1) {
                               rr = rr_first = t0;
                               bb = t1;
                               active = bb > 0.0;
                               flags = active ? 0 : kFlagConverged;
                               check();
                               return 0.0;
                           },
                           beta, any))
            return give_up();
        for (;;) {
            while (any && it < A.max_steps) {  // (the same in every thread of the group)
                ++it;
                // A
                clear();
#pragma unroll
                for (int l = 0; l < WG; ++l) {
                    double2 t[NC];
                    gather(Rk(cur), yo, l, t);
#pragma unroll
                    for (int b = 0; b < NC; ++b) {
                        pn[l][b].x = fma(beta[l], pn[l][b].x, t[b].x);
                        pn[l][b].y = fma(beta[l], pn[l][b].y, t[b].y);
                    }
                    const double g = hop_sum(ho, pn[l]);
                    p[l] = fma(beta[l], p[l], r[l]);
                    if (EO) {
                        const double po = ic * g;
                        publish(Wk(cur), l, po);
                        v[2 * l] = p[l] * p[l];
                        v[2 * l + 1] = own ? po * po : 0.0;
                    } else {
                        q[l] = fma(c, p[l], -g);
                        v[2 * l] = own ? p[l] * q[l] : 0.0;
                    }
                }
                double alpha[WG];
                if (!small_sum<WG>(A, sh, polls, tag, v, active,
                                   [&](double t0, double t1) {
                                       const double pq = EO ? c * (t0 - t1) : t0;
                                       if (!active) return 0.0;
                                       if (!(pq > 0.0) || !isfinite(pq)) {
                                           active = 0;
                                           if (!A.refine) flags |= kFlagBreakdown;
                                           return 0.0;
                                       }
                                       ++iters;
                                       return rr / pq;
                                   },
                                   alpha, any))
                    return give_up();
                // B
                const int next = cur + 1 < A.nring ? cur + 1 : 0;
                clear();
#pragma unroll
                for (int l = 0; l < WG; ++l) {
                    if (EO) {
                        double2 t[NC];
                        gather(Wk(cur), ye, l, t);
                        q[l] = fma(c, p[l], -hop_sum(he, t));
                    }
                    if (own) {
                        r[l] = fma(-alpha[l], q[l], r[l]);
                        x[l] = fma(alpha[l], p[l], x[l]);
                    }
                    publish(Rk(next), l, r[l]);
                    v[2 * l] = r[l] * r[l];
                }
                if (!small_sum<WG>(A, sh, polls, tag, v, active,
                                   [&](double t0, double) {
                                       if (!active) return 0.0;
                                       const double f = t0 / rr;
                                       rr = t0;
                                       check();
                                       return active ? f : 0.0;
                                   },
                                   beta, any))
                    return give_up();
                advance();
            }
            // the odd half of x, then the true residual; x_e takes the place
            // of the r that no one has read
#pragma unroll
            for (int l = 0; l < WG; ++l) publish(Rk(cur), l, x[l]);
            clear();
            if (!small_sum<WG>(A, sh, polls, tag, v, active, none, out, any)) return give_up();
            if (EO) {
#pragma unroll
                for (int l = 0; l < WG; ++l) {
                    double2 t[NC];
                    gather(Rk(cur), yo, l, t);
                    const double g = hop_sum(ho, t);
                    const double xo = ic * (b_own(ns + s, l) + g);
                    publish(Wk(cur), l, xo);
                    if (own && l0 + l < A.W) A.x[2 * ((size_t)((ns + s) * NC + ca) * A.W + l0 + l) + im] = xo;
                }
                if (!small_sum<WG>(A, sh, polls, tag, v, active, none, out, any)) return give_up();
            }
            const int next = cur + 1 < A.nring ? cur + 1 : 0;
#pragma unroll
            for (int l = 0; l < WG; ++l) {
                double2 t[NC];
                gather(EO ? Wk(cur) : Rk(cur), ye, l, t);
                const double g = hop_sum(he, t);
                const double rt = own ? b_own(s, l) - fma(c, x[l], -g) : 0.0;
                v[2 * l] = rt * rt;
                if (A.refine) {
                    r[l] = rt;
                    publish(Rk(next), l, rt);
                }
            }
            ++nref;
            if (!small_sum<WG>(A, sh, polls, tag, v, active,
                               [&](double t0, double) {
                                   true_rr = t0;
                                   if (!A.refine) {
                                       active = 0;  // (done; flags and iters stay)
                                       return 0.0;
                                   }
                                   // the true residual decides: a lane that misses the tolerance goes on
                                   rr = t0;
                                   if (t0 <= cs.tol2 * bb) {
                                       flags |= kFlagConverged;
                                       active = 0;
                                   } else if (flags & kFlagConverged) {
                                       flags &= ~kFlagConverged;
                                       active = 1;
                                   }
                                   return 0.0;
                               },
                               beta, any))
                return give_up();
            advance();
            if (!any || it >= A.max_steps) break;
        }
#pragma unroll
        for (int l = 0; l < WG; ++l)
            if (own && l0 + l < A.W) A.x[2 * ((size_t)(s * NC + ca) * A.W + l0 + l) + im] = x[l];
        if (wb == 0 && tid < WG && l0 + tid < A.W) {
            const int j = l0 + tid;
            cs.rr[j] = rr;
            cs.qp[j] = 0.0;
            cs.rr_ref[j] = rr_first;
            cs.bb[j] = bb;
            cs.alpha[j] = 0.0;
            cs.beta[j] = 0.0;
            cs.true_rr[j] = true_rr;
            cs.active[j] = active;
            cs.iters[j] = iters;
            cs.flags[j] = flags;
            if (j == 0) *A.nref = A.refine ? nref : 0;
        }
    }
}

// ============================================================ deflation
//
// Dense pieces of the deflated estimator (Sec. Deflation) on blocks of FP64
// vectors in the internal layout, read as row-major matrices [n rows =
// N * nc][width] (width = the block's lanes).

// t_j = sum_x sum_b conj(u_j(x,b)) w_j(x + p e0, b)
__global__ __launch_bounds__(kBlock) void k_dot_shift(Launch L, const double2 *__restrict__ u,
                                                      const double2 *__restrict__ w, int p, Red rd) {
    __shared__ double sm[2 * kBlock];
    const int tid = threadIdx.x, logW = L.logW, W = L.W;
    const int j = tid & (W - 1), sl = tid >> logW;
    const int sites_per_tile = kBlock >> logW, nc = L.nc;
    double acc[2] = {0.0, 0.0};
    int t0, t1;
    const Blk bk = own_blk();
    tile_range(bk, L.ntiles, t0, t1);
    for (int t = t0; t < t1; ++t) {
        const int site = t * sites_per_tile + sl;
        if (site >= L.lat.N) continue;
        const int y = shift0(L.lat, site, p);
        for (int b = 0; b < nc; ++b) {
            const double2 a = u[((size_t)(site * nc + b) << logW) + j];
            const double2 c = w[((size_t)(y * nc + b) << logW) + j];
            acc[0] += a.x * c.x + a.y * c.y;
            acc[1] += a.x * c.y - a.y * c.x;
        }
    }
    block_partials<2>(bk, acc, W, logW, rd, sm);
}

// per-lane |u_j - theta_j w_j|^2 (Ritz residuals: u = A v, w = v)
__global__ __launch_bounds__(kBlock) void k_resid_norm(Launch L, const double2 *__restrict__ u,
                                                       const double2 *__restrict__ w,
                                                       const double *__restrict__ theta, Red rd) {
    __shared__ double sm[kBlock];
    const int tid = threadIdx.x, W = L.W;
    const int sites_per_tile = kBlock >> L.logW;
    const double th = theta[tid & (W - 1)];
    double acc[1] = {0.0};
    int t0, t1;
    const Blk bk = own_blk();
    tile_range(bk, L.ntiles, t0, t1);
    const size_t e0 = (size_t)t0 * sites_per_tile * L.nc * W;
    const size_t e1 = min((size_t)t1 * sites_per_tile, (size_t)L.lat.N) * L.nc * W;
    for (size_t e = e0 + tid; e < e1; e += kBlock) {
        const double2 a = u[e], c = w[e];
        const double dr = a.x - th * c.x, di = a.y - th * c.y;
        acc[0] += dr * dr + di * di;
    }
    block_partials<1>(bk, acc, W, L.logW, rd, sm);
}

// out = a q + b v (real a, b; out may alias v)
__global__ void k_axpby(long long n, double a, const double2 *__restrict__ q, double b, const double2 *v,
                        double2 *out) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const double2 x = q[e], y = v[e];
    out[e] = make_double2(a * x.x + b * y.x, a * x.y + b * y.y);
}

// v[e] = (+-1 +- i) from a SplitMix64 hash of (seed, e): start vectors of
// the subspace iteration
__global__ void k_rand_fill(long long n, unsigned long long seed, double2 *__restrict__ v) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const unsigned long long h = mix64(mix64(seed) ^ (unsigned long long)e);
    v[e] = make_double2((h >> 63) ? -1.0 : 1.0, ((h >> 62) & 1) ? -1.0 : 1.0);
}

// out lane j = v lane j * s[j] (s[j] = 0 clears the lane)
__global__ void k_scale_lanes(long long n, int W, const double *__restrict__ s, const double2 *__restrict__ v,
                              double2 *__restrict__ out) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n) return;
    const double f = s[e % W];
    const double2 x = v[e];
    out[e] = make_double2(f * x.x, f * x.y);
}

// Partial products H = X^H Y over one range of rows per workgroup (blockIdx.x)
// for one 32 x 32 output tile (blockIdx.y): part[blockIdx.x][blockIdx.y][32 * 32].
// A contraction over the rows, on the FP64 matrix instruction (16 x 16 outputs,
// four rows): lane l of a wavefront supplies column l % 16 of row l / 16 of either
// operand, which is how it loads them (whole 256-byte rows of 16 columns), so
// there is no LDS tile and no barrier per stage, and X and Y are all that is
// moved.  The wavefronts take 16 rows each in turn; their sums meet in order.
// (64 x 64 tiles staged through LDS, 16 outputs per thread, padded 16 x 32
// outputs to 64 x 64: n = 196608, 16 x 32: 374 us, 24 now (the vectors partly in the
// Infinity Cache).)
constexpr int kGramTile = 32;
typedef double f64x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kBlock) void k_gram(long long n, int WX, int WY, const double2 *__restrict__ X,
                                                 const double2 *__restrict__ Y, double2 *__restrict__ part) {
    __shared__ double2 sum[kGramTile * kGramTile];
    const int tilesY = (WY + kGramTile - 1) / kGramTile;
    const int i0 = (blockIdx.y / tilesY) * kGramTile, j0 = (blockIdx.y % tilesY) * kGramTile;
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, c = lane & 15, k = lane >> 4;
    const int ni = i0 + 16 < WX ? 2 : 1, nj = j0 + 16 < WY ? 2 : 1;  // 16-wide halves in use
    f64x4 re[2][2] = {}, im[2][2] = {};
    const long long r0 = n * blockIdx.x / gridDim.x, r1 = n * (blockIdx.x + 1) / gridDim.x;
    for (long long rb = r0 + 16 * wave; rb < r1; rb += 16 * (kBlock / 64)) {
        double2 x[4][2], y[4][2];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const long long r = rb + 4 * q + k;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int ci = i0 + 16 * h + c, cj = j0 + 16 * h + c;
                x[q][h] = y[q][h] = make_double2(0.0, 0.0);
                if (r < r1 && ci < WX) x[q][h] = ldg(X + r * WX + ci);
                if (r < r1 && cj < WY) y[q][h] = ldg(Y + r * WY + cj);
            }
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int g = 0; g < 2; ++g) {
                    if (h >= ni || g >= nj) continue;
                    // conj(x) y
                    re[h][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[q][h].x, y[q][g].x, re[h][g], 0, 0, 0);
                    re[h][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[q][h].y, y[q][g].y, re[h][g], 0, 0, 0);
                    im[h][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[q][h].x, y[q][g].y, im[h][g], 0, 0, 0);
                    im[h][g] = __builtin_amdgcn_mfma_f64_16x16x4f64(-x[q][h].y, y[q][g].x, im[h][g], 0, 0, 0);
                }
    }
    // entry v of a lane's result: row 4 v + l / 16, column l % 16
    for (int w = 0; w < kBlock / 64; ++w) {
        if (wave == w)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int g = 0; g < 2; ++g)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        double2 &o = sum[(16 * h + 4 * v + k) * kGramTile + 16 * g + c];
                        const double2 a = w ? o : make_double2(0.0, 0.0);
                        o = make_double2(a.x + re[h][g][v], a.y + im[h][g][v]);
                    }
        __syncthreads();
    }
    double2 *o = part + ((size_t)blockIdx.x * gridDim.y + blockIdx.y) * kGramTile * kGramTile;
    for (int e = t; e < kGramTile * kGramTile; e += kBlock) o[e] = sum[e];
}

// H[i][j] = scale * the sum of the partials over the row ranges: 16 entries per
// workgroup, 16 threads to an entry (thread g adds ranges g, g + 16, ...), then
// those in order.  (One thread per entry: 74 us for 256 ranges of 16 x 32, now
// below 9.)
__global__ __launch_bounds__(kBlock) void k_gram_reduce(int nrb, int WX, int WY, const double2 *__restrict__ part,
                                                        double scale, double2 *__restrict__ H) {
    __shared__ double2 sums[16][16];
    const int c = threadIdx.x & 15, g = threadIdx.x >> 4;
    const int e = blockIdx.x * 16 + c;
    double sr = 0.0, si = 0.0;
    if (e < WX * WY) {
        const int i = e / WY, j = e % WY;
        const int tilesY = (WY + kGramTile - 1) / kGramTile;
        const int tiles = ((WX + kGramTile - 1) / kGramTile) * tilesY;
        const int tile = (i / kGramTile) * tilesY + j / kGramTile;
        const int off = (i % kGramTile) * kGramTile + j % kGramTile;
        for (int b = g; b < nrb; b += 16) {
            const double2 v = part[((size_t)b * tiles + tile) * kGramTile * kGramTile + off];
            sr += v.x;
            si += v.y;
        }
    }
    sums[g][c] = make_double2(sr, si);
    __syncthreads();
    if (g != 0 || e >= WX * WY) return;
    for (int q = 1; q < 16; ++q) {
        sr += sums[q][c].x;
        si += sums[q][c].y;
    }
    H[e] = make_double2(scale * sr, scale * si);
}

// out[r][j] (+)= sum_i X[r][i] C[i][j], j < WY, i < WX (out must not alias X)
__global__ void k_rot(long long n, int WX, int WY, const double2 *__restrict__ X, const double2 *__restrict__ C,
                      double2 *__restrict__ out, int accumulate) {
    const long long e = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= n * WY) return;
    const long long r = e / WY;
    const int j = (int)(e - r * WY);
    double sr = 0.0, si = 0.0;
    if (accumulate) {
        sr = out[e].x;
        si = out[e].y;
    }
    const double2 *xr = X + r * WX;
    for (int i = 0; i < WX; ++i) {
        const double2 x = xr[i], c = C[(size_t)i * WY + j];
        sr = fma(x.x, c.x, fma(-x.y, c.y, sr));
        si = fma(x.x, c.y, fma(x.y, c.x, si));
    }
    out[e] = make_double2(sr, si);
}

// per-site bound sum over the eight hops of |U|_F (FP64 hop links)
__global__ void k_hop_bound(Lat lat, int nc, const double2 *__restrict__ U8, double *__restrict__ out) {
    const int site = blockIdx.x * blockDim.x + threadIdx.x;
    if (site >= lat.N) return;
    double s = 0.0;
    for (int d = 0; d < 8; ++d) {
        double f = 0.0;
        for (int e = 0; e < nc * nc; ++e) {
            const double2 u = U8[((size_t)site * 8 + d) * nc * nc + e];
            f += u.x * u.x + u.y * u.y;
        }
        s += sqrt(f);
    }
    out[site] = s;
}

// ============================================================ launchers

static int blocks_for(long long n) { return (int)((n + kBlock - 1) / kBlock); }

int grid_blocks(int ntiles) {
    // four workgroups per CU, a multiple of 8 (one contiguous share per
    // XCD); never more than there are tiles.  All of them are resident at
    // once, so they walk their slabs in step (16^4 sites, FP32, W = 32: a
    // CG iteration took 3% less time than with 2048, 14% less than with 512)
    const int cap = 1024;
    if (ntiles <= 8) return ntiles;
    int n = ntiles < cap ? ntiles : cap;
    return n - n % 8;
}

void prepare_links(const Lat &lat, int nc, const void *abi, int *nbr, double *u64, int prec, void *u8,
                   double *u8x, hipStream_t s) {
    const long long n = 8LL * lat.N * (abi ? nc * nc : 1);
    const double2 *in = (const double2 *)abi;
    if (prec == kF64)
        k_prepare<double2><<<blocks_for(n), kBlock, 0, s>>>(lat, nc, in, nbr, (double2 *)u64, (double2 *)u8,
                                                            (double2 *)u8x);
    else if (prec == kF32)
        k_prepare<float2><<<blocks_for(n), kBlock, 0, s>>>(lat, nc, in, nbr, (double2 *)u64, (float2 *)u8,
                                                           (double2 *)u8x);
    else
        k_prepare<bf16x2><<<blocks_for(n), kBlock, 0, s>>>(lat, nc, in, nbr, (double2 *)u64, (bf16x2 *)u8,
                                                           (double2 *)u8x);
}

#define DP_DISPATCH_PREC(prec, S, ...)          \
    do {                                        \
        if ((prec) == kF64) {                   \
            using S = double2;                  \
            __VA_ARGS__;                        \
        } else if ((prec) == kF32) {            \
            using S = float2;                   \
            __VA_ARGS__;                        \
        } else {                                \
            using S = bf16x2;                   \
            __VA_ARGS__;                        \
        }                                       \
    } while (0)

template <int SRC>
static void init_block(const Launch &L, int prec, const ProbeGen &g, const double *src, long long rhs0,
                       long long nvalid, const InitArgs &ia) {
    DP_DISPATCH_PREC(prec, S,
                     k_init<S, SRC><<<L.nblk, kBlock, 0, L.stream>>>(L, g, (const double2 *)src, rhs0, nvalid,
                                                                     (double2 *)ia.b64, (S *)ia.r, (S *)ia.p,
                                                                     (S *)ia.xlo, 1.0 / ia.diag, ia.rd));
    if (!L.lat.eo) {
        k_finish<2, kEpiInit><<<L.W, kBlock, 0, L.stream>>>(ia.rd, ia.cs);
        return;
    }
    // r = p = b_e + H b_o / c: the odd half of p holds -b_o / c
    StencilArgs a;
    a.kind = kStInit;
    a.links = ia.links;
    a.diag = 1.0;
    a.pin = ia.p;
    a.q = ia.r;
    a.q2 = ia.p;
    a.U = ia.U;
    a.nbr = ia.nbr;
    a.cg = 1;
    a.rd = ia.rd;
    a.cs = ia.cs;
    launch_stencil(L, prec, a);
}

template <typename S, int NC, bool LINKS>
static void init_probe_t(const Launch &L, const ProbeGen &g, const InitArgs &ia) {
    k_init_probe<S, NC, LINKS><<<L.nblk, kBlock, 0, L.stream>>>(L, g, (S *)ia.r, (S *)ia.p, (S *)ia.xlo,
                                                                1.0 / ia.diag, (const double2 *)ia.U64, ia.rd);
}

void launch_init_probe(const Launch &L, int prec, const ProbeGen &g, const InitArgs &ia) {
    if (!L.lat.eo) {
        init_block<0>(L, prec, g, nullptr, 0, 0, ia);
        return;
    }
    DP_DISPATCH_PREC(prec, S, {
        if (L.nc == 3)
            ia.links ? init_probe_t<S, 3, true>(L, g, ia) : init_probe_t<S, 3, false>(L, g, ia);
        else
            ia.links ? init_probe_t<S, 1, true>(L, g, ia) : init_probe_t<S, 1, false>(L, g, ia);
    });
    k_finish<4, kEpiInitEo><<<L.W, kBlock, 0, L.stream>>>(ia.rd, ia.cs);
}

void launch_init_abi(const Launch &L, int prec, const double *babi, long long rhs0, long long nvalid,
                     const InitArgs &ia) {
    init_block<1>(L, prec, ProbeGen{}, babi, rhs0, nvalid, ia);
}

// Stencil modes a launch shape admits.  The grouped modes need the slab walk
// (a grid of a multiple of 8 workgroups over x0-slabs): pairs an even
// number of slices per slab, quads two slices and an even D3, lines a
// multiple of four slices; the LDS tiles take W >= 16 (pairs, mode 1) or
// W >= 32 (quads, lines); mode 2 a wavefront per site (W >= 64); mode 5
// one right-hand side (not BF16).
bool stencil_mode_valid(const Launch &L, int prec, int mode) {
    // (the grouped modes' members are neighbours in the index order)
    const bool slabs = L.nblk >= 8 && L.nblk % 8 == 0 && L.lat.D[0] % 8 == 0 && !L.lat.eo;
    const int n0 = L.lat.D[0] / 8;
    switch (mode) {
        case 0: return true;
        case 1: return L.W >= 16;
        case 2: return L.W >= 64;
        case 3: return slabs && n0 % 2 == 0 && L.W >= 16;
        case 4: return slabs && n0 == 2 && L.lat.D[3] % 2 == 0 && L.W >= 32;
        case 5: return L.W == 1 && prec != kBF16;
        case 6: return slabs && n0 % 4 == 0 && L.W >= 32;
        default: return false;
    }
}

// The choice without timing: the grouped modes where they apply (not for
// BF16, whose packed-dot body has none), else by width.
int stencil_mode_rule(const Launch &L, int prec) {
    const bool bf = prec == kBF16;
    if (L.W == 1 && !bf) return 5;
    if (L.W >= 64) return 2;
    if (!bf && stencil_mode_valid(L, prec, 4)) return 4;
    if (!bf && stencil_mode_valid(L, prec, 6)) return 6;
    if (!bf && stencil_mode_valid(L, prec, 3)) return 3;
    return L.W >= 16 ? 1 : 0;
}

template <typename S, typename LS, int NC, bool LINKS, int KIND>
static void stencil_nc(const Launch &L, const StencilArgs &a) {
    using R = typename St<S>::R;
    dim3 grid(L.nblk), blk(kBlock);
    const S *pin = (const S *)a.pin, *rin = (const S *)a.rin;
    S *q = (S *)a.q, *q2 = (S *)a.q2;
    const LS *U = (const LS *)a.U;
    HopB hb{(const double2 *)a.b64, a.gen ? *a.gen : ProbeGen{}, a.gen ? 1 : 0};
#define DP_ST(M)                                                                                              \
    if (a.ev0)                                                                                                \
        hipExtLaunchKernelGGL(k_stencil<S, LS, NC, LINKS, M, KIND>, grid, blk, 0, L.stream, a.ev0, a.ev1, 0, L, \
                              (R)a.diag, pin, rin, q, q2, U, a.nbr, a.cg, a.rd, hb);                          \
    else                                                                                                      \
        k_stencil<S, LS, NC, LINKS, M, KIND><<<grid, blk, 0, L.stream>>>(L, (R)a.diag, pin, rin, q, q2, U, a.nbr, \
                                                                         a.cg, a.rd, hb)
    constexpr int prec = std::is_same<S, double2>::value ? kF64 : (std::is_same<S, float2>::value ? kF32 : kBF16);
    if constexpr (KIND == kStHopB) {  // (W = 1: see stencil_kind)
        DP_ST(5);
        return;
    }
    const int mode = L.smode >= 0 && stencil_mode_valid(L, prec, L.smode) ? L.smode : stencil_mode_rule(L, prec);
    switch (mode) {
        case 5:
            if constexpr (prec != kBF16) {
                DP_ST(5);
                break;
            }
            [[fallthrough]];
        case 0: DP_ST(0); break;
        case 1: DP_ST(1); break;
        case 2: DP_ST(2); break;
        default:  // the grouped modes: never in even-odd order
            if constexpr (KIND == kStFull) {
                if (mode == 3) {
                    DP_ST(3);
                } else if (mode == 4) {
                    DP_ST(4);
                } else {
                    DP_ST(6);
                }
            }
            break;
    }
#undef DP_ST
}

template <typename S, typename LS, int KIND>
static void stencil_t(const Launch &L, const StencilArgs &a) {
    if (L.nc == 3) {
        if (a.links)
            stencil_nc<S, LS, 3, true, KIND>(L, a);
        else
            stencil_nc<S, LS, 3, false, KIND>(L, a);
    } else {
        if (a.links)
            stencil_nc<S, LS, 1, true, KIND>(L, a);
        else
            stencil_nc<S, LS, 1, false, KIND>(L, a);
    }
}

// The odd half of the solution (W > 1; the modes go by width as the stencil's)
template <int NC, bool LINKS>
static void odd_x_t(const Launch &L, const StencilArgs &a) {
    const ProbeGen g = a.gen ? *a.gen : ProbeGen{};
#define DP_OX(M)                                                                                                   \
    k_odd_x<NC, LINKS, M><<<L.nblk, kBlock, 0, L.stream>>>(L, a.diag, (const double2 *)a.b64, (double2 *)a.q,      \
                                                           (const double2 *)a.U, a.nbr, g, a.gen ? 1 : 0)
    if (L.W >= 64)
        DP_OX(2);
    else if (L.W >= 16)
        DP_OX(1);
    else
        DP_OX(0);
#undef DP_OX
}

static void odd_x(const Launch &L, const StencilArgs &a) {
    if (L.nc == 3)
        a.links ? odd_x_t<3, true>(L, a) : odd_x_t<3, false>(L, a);
    else
        a.links ? odd_x_t<1, true>(L, a) : odd_x_t<1, false>(L, a);
}

template <typename S>
static void stencil_kind(const Launch &L, const StencilArgs &a) {
    if (a.kind == kStHop) return stencil_t<S, S, kStHop>(L, a);
    if (a.kind == kStInit) return stencil_t<S, S, kStInit>(L, a);
    if constexpr (std::is_same<S, double2>::value)
        if (a.kind == kStHopB) return L.W == 1 ? stencil_t<S, S, kStHopB>(L, a) : odd_x(L, a);
    stencil_t<S, S, kStFull>(L, a);
}

void launch_stencil(const Launch &L, int prec, const StencilArgs &a) {
    DP_DISPATCH_PREC(prec, S, stencil_kind<S>(L, a));
    if (a.kind == kStInit)
        k_finish<4, kEpiInitEo><<<L.W, kBlock, 0, L.stream>>>(a.rd, a.cs);
    else if (a.cg)
        k_finish_cg<<<L.W, kBlock, 0, L.stream>>>(a.rd, a.cs);
}

template <typename S, int XNT>
static void update_t(const Launch &L, void *x, void *r, void *p, const void *q, const Red &rd, const CgState &cs,
                     int xmode) {
    if constexpr (!std::is_same<S, double2>::value) {
        if (xmode == 1)
            return k_update<S, 1, XNT><<<L.nblk, kBlock, 0, L.stream>>>(L, (S *)x, (S *)r, (S *)p, (const S *)q, rd,
                                                                        cs);
        if (xmode == 2)
            return k_update<S, 2, XNT><<<L.nblk, kBlock, 0, L.stream>>>(L, (S *)x, (S *)r, (S *)p, (const S *)q, rd,
                                                                        cs);
    }
    k_update<S, 0, XNT><<<L.nblk, kBlock, 0, L.stream>>>(L, (S *)x, (S *)r, (S *)p, (const S *)q, rd, cs);
}

void launch_update(const Launch &L, int prec, void *x, void *r, void *p, const void *q, const Red &rd,
                   const CgState &cs, int xmode) {
    if (!cs.xdef) xmode = 0;  // (deferral: FP32 and BF16 storage)
    DP_DISPATCH_PREC(prec, S,
                     L.xnt == 0   ? update_t<S, 0>(L, x, r, p, q, rd, cs, xmode)
                     : L.xnt == 1 ? update_t<S, 1>(L, x, r, p, q, rd, cs, xmode)
                                  : update_t<S, 2>(L, x, r, p, q, rd, cs, xmode));
}

void launch_fold(const Launch &L, int prec, double *x64, void *xlo, int first) {
    DP_DISPATCH_PREC(prec, S, k_fold<S><<<L.nblk, kBlock, 0, L.stream>>>(L, (double2 *)x64, (S *)xlo, first));
}

template <typename S, int NC, bool LINKS>
static void true_resid_t(const Launch &L, const ResidArgs &a) {
    const ProbeGen g = a.gen ? *a.gen : ProbeGen{};
#define DP_TR(M)                                                                                                  \
    k_true_resid<S, NC, LINKS, M><<<L.nblk, kBlock, 0, L.stream>>>(                                               \
        L, a.diag, (const double2 *)a.b64, (const double2 *)a.x64, (const double2 *)a.U64, a.nbr, (S *)a.r, (S *)a.p, \
        (const S *)a.q, a.ru, a.rd, a.cs, g, a.gen ? 1 : 0)
    // (by width as the stencil's; at W = 64 the LDS tile took the fine trace of
    // 16^4 x 3, FP32, from 167 to 171 ms)
    if (L.W >= 64)
        DP_TR(2);
    else if (L.W >= 16)
        DP_TR(1);
    else
        DP_TR(0);
#undef DP_TR
}

void launch_true_resid(const Launch &L, int prec, const ResidArgs &a) {
    DP_DISPATCH_PREC(prec, S, {
        if (L.nc == 3)
            a.links ? true_resid_t<S, 3, true>(L, a) : true_resid_t<S, 3, false>(L, a);
        else
            a.links ? true_resid_t<S, 1, true>(L, a) : true_resid_t<S, 1, false>(L, a);
    });
    if (a.ru)
        k_finish<2, kEpiRU><<<L.W, kBlock, 0, L.stream>>>(a.rd, a.cs);
    else
        k_finish<2, kEpiStats><<<L.W, kBlock, 0, L.stream>>>(a.rd, a.cs);
}

void launch_resid_q(const Launch &L, int prec, const double *b64, const double *q64, void *r, void *p,
                    const void *q, int ru_mode, const Red &rd, const CgState &cs, const ProbeGen *gen) {
    const ProbeGen g = gen ? *gen : ProbeGen{};
    const int use_gen = gen ? 1 : 0;
    const double2 *b = (const double2 *)b64, *qq = (const double2 *)q64;
    DP_DISPATCH_PREC(prec, S, {
        if (L.nc == 3)
            k_resid_q<S, 3><<<L.nblk, kBlock, 0, L.stream>>>(L, b, qq, (S *)r, (S *)p, (const S *)q, ru_mode, rd, cs,
                                                             g, use_gen);
        else
            k_resid_q<S, 1><<<L.nblk, kBlock, 0, L.stream>>>(L, b, qq, (S *)r, (S *)p, (const S *)q, ru_mode, rd, cs,
                                                             g, use_gen);
    });
    if (ru_mode)
        k_finish<2, kEpiRU><<<L.W, kBlock, 0, L.stream>>>(rd, cs);
    else
        k_finish<2, kEpiStats><<<L.W, kBlock, 0, L.stream>>>(rd, cs);
}

void launch_level_map(int N, const int *fine, int nfine, const int *coarse, int ncoarse, int *cmap, int *bad,
                      hipStream_t s) {
    k_level_map_clear<<<blocks_for(nfine), kBlock, 0, s>>>(cmap, nfine, bad);
    k_level_map_scatter<<<blocks_for(N), kBlock, 0, s>>>(N, fine, nfine, coarse, ncoarse, cmap, bad);
    k_level_map_check<<<blocks_for(N), kBlock, 0, s>>>(N, fine, nfine, coarse, cmap, bad);
}

void launch_displaced_dot(const Launch &L, const ProbeGen &g, int p, const double *x64, const Red &rd,
                          const CgState &cs) {
    k_displaced_dot<<<L.nblk, kBlock, 0, L.stream>>>(L, g, p, (const double2 *)x64, rd, cs);
    k_finish<2, kEpiTj><<<L.W, kBlock, 0, L.stream>>>(rd, cs);
}

void launch_dot(const Launch &L, const double *a64, const double *b64, const Red &rd, const CgState &cs) {
    k_dot<<<L.nblk, kBlock, 0, L.stream>>>(L, (const double2 *)a64, (const double2 *)b64, rd, cs);
    k_finish<2, kEpiTj><<<L.W, kBlock, 0, L.stream>>>(rd, cs);
}

void launch_ctrl(const Red &rd, const CgState &cs, int W, hipStream_t s) {
    k_finish<2, kEpiCheck><<<W, kBlock, 0, s>>>(rd, cs);
    k_ctrl<<<1, 64, 0, s>>>(cs, W);
}

// The same force for W >= 8, W threads per (site, mu) pair: thread j loads
// lane j of the four rows the pair needs (coalesced, each once per pair) and
// forms its lane's 4 nc^2 doubles (padded to 8 * 5 = 40 for nc = 3); the
// lanes are summed by a reduce-scatter inside the wavefront (three halvings:
// a lane keeps one half of its values and adds its partner's copy of that
// half, so the shuffles move 20 + 10 + 5 values instead of 3 x 40), a
// butterfly on the remaining five, and through LDS across the wavefronts of
// a pair (W > 64); all in a fixed order.
template <int NC>
__global__ __launch_bounds__(kBlock) void k_force_lanes(Launch L, const double2 *__restrict__ x64,
                                                        const double2 *__restrict__ l64, const int *__restrict__ nbr,
                                                        double scale, int first, double *__restrict__ dU,
                                                        double *__restrict__ dUbar) {
    constexpr int NV = 4 * NC * NC;         // dU re, dU im, dUbar re, dUbar im per (a, b)
    constexpr int NP = (NV + 7) / 8 * 8;    // padded so that three halvings divide it
    __shared__ double red[kBlock / 8][NP];  // one row per pair (W < 64) or per wavefront (W >= 64)
    const int W = L.W, logW = L.logW, tid = threadIdx.x;
    const int j = tid & (W - 1), pl = tid >> logW;
    const long long pair = (long long)blockIdx.x * (kBlock >> logW) + pl;
    const bool live = pair < (long long)L.lat.N * 4;
    const int site = live ? (int)(pair >> 2) : 0, mu = (int)(pair & 3);
    double v[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) v[k] = 0.0;
    if (live) {
        const int y = nbr[site * 8 + mu];
        double2 la[NC], xa[NC], xb[NC], lb[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            la[c] = l64[((size_t)(site * NC + c) << logW) + j];
            xa[c] = x64[((size_t)(site * NC + c) << logW) + j];
            xb[c] = x64[((size_t)(y * NC + c) << logW) + j];
            lb[c] = l64[((size_t)(y * NC + c) << logW) + j];
        }
#pragma unroll
        for (int a = 0; a < NC; ++a)
#pragma unroll
            for (int b = 0; b < NC; ++b) {
                const int k = 4 * (a * NC + b);
                v[k] = la[a].x * xb[b].x + la[a].y * xb[b].y;  // conj(l) x
                v[k + 1] = la[a].x * xb[b].y - la[a].y * xb[b].x;
                v[k + 2] = xa[a].x * lb[b].x + xa[a].y * lb[b].y;  // x conj(l)
                v[k + 3] = xa[a].y * lb[b].x - xa[a].x * lb[b].y;
            }
    }
    // reduce-scatter over the span = min(W, 64) lanes of a group (W >= 8:
    // three halvings fit), then a butterfly over the rest of the span
    const int span = W < 64 ? W : 64, lane = tid & 63;
    int base = 0;  // first value this lane holds after the halvings
#pragma unroll
    for (int step = 0; step < 3; ++step) {
        const int off = span >> (step + 1);
        const int half = NP >> (step + 1);
        const bool upper = (lane & off) != 0;
#pragma unroll
        for (int k = 0; k < half; ++k) {
            const double keep = upper ? v[k + half] : v[k];
            const double give = upper ? v[k] : v[k + half];
            v[k] = keep + __shfl_xor(give, off, 64);
        }
        base += upper ? half : 0;
    }
    constexpr int NR = NP / 8;  // values per lane after the halvings
    for (int off = span >> 4; off > 0; off >>= 1)
#pragma unroll
        for (int k = 0; k < NR; ++k) v[k] += __shfl_xor(v[k], off, 64);
    // lanes with the low bits of the span clear hold the sums of their values
    const int row = W < 64 ? pl : (tid >> 6);
    if ((lane & ((span >> 3) - 1)) == 0)
#pragma unroll
        for (int k = 0; k < NR; ++k) red[row][base + k] = v[k];
    __syncthreads();
    if (!live) return;
    const int nw = W < 64 ? 1 : W >> 6, r0 = W < 64 ? pl : (pl * W) >> 6, x = lex_of(L.lat, site);
    for (int k = j; k < NV; k += W) {
        double t = red[r0][k];
        for (int w = 1; w < nw; ++w) t += red[r0 + w][k];
        const int ab = k >> 2, comp = k & 3;
        const size_t o = 2 * (((size_t)mu * L.lat.N + x) * NC * NC + ab) + (comp & 1);
        double *out = comp < 2 ? dU : dUbar;
        if (!out) continue;
        t *= scale;
        out[o] = first ? t : out[o] + t;
    }
}

void launch_force(const Launch &L, const double *x64, const double *l64, const int *nbr, double scale, int first,
                  double *dU, double *dUbar) {
    if (L.W >= 8) {
        // W threads per (site, mu) pair
        const long long nthreads = (long long)L.lat.N * 4 * L.W;
        if (L.nc == 3)
            k_force_lanes<3><<<blocks_for(nthreads), kBlock, 0, L.stream>>>(L, (const double2 *)x64,
                                                                           (const double2 *)l64, nbr, scale, first,
                                                                           dU, dUbar);
        else
            k_force_lanes<1><<<blocks_for(nthreads), kBlock, 0, L.stream>>>(L, (const double2 *)x64,
                                                                           (const double2 *)l64, nbr, scale, first,
                                                                           dU, dUbar);
        return;
    }
    const long long n = (long long)L.lat.N * 4 * L.nc * L.nc;
    k_force<<<blocks_for(n), kBlock, 0, L.stream>>>(L, (const double2 *)x64, (const double2 *)l64, nbr, scale,
                                                    first, (double2 *)dU, (double2 *)dUbar);
}

template <int NC, bool LINKS, bool EO>
static void small_t(const SmallArgs &a, hipStream_t s) {
    const int grid = a.nwg * a.ngroups;
    switch (a.wg) {
        case 1: k_small<NC, LINKS, EO, 1><<<grid, kSmallThreads, 0, s>>>(a); break;
        case 2: k_small<NC, LINKS, EO, 2><<<grid, kSmallThreads, 0, s>>>(a); break;
        default: k_small<NC, LINKS, EO, 4><<<grid, kSmallThreads, 0, s>>>(a); break;
    }
}

void launch_small(const SmallArgs &a, hipStream_t s) {
    if (a.nc == 3) {
        if (a.links)
            a.lat.eo ? small_t<3, true, true>(a, s) : small_t<3, true, false>(a, s);
        else
            a.lat.eo ? small_t<3, false, true>(a, s) : small_t<3, false, false>(a, s);
    } else {
        if (a.links)
            a.lat.eo ? small_t<1, true, true>(a, s) : small_t<1, true, false>(a, s);
        else
            a.lat.eo ? small_t<1, false, true>(a, s) : small_t<1, false, false>(a, s);
    }
}

void launch_small_clear(unsigned long long *part, hipStream_t s) {
    static_assert(kSmallPartBytes % (8 * kBlock) == 0, "whole workgroups of words");
    k_small_clear<<<kSmallPartBytes / (8 * kBlock), kBlock, 0, s>>>(part);
}

void launch_small_go(unsigned *stop, hipStream_t s) { k_small_go<<<1, 1, 0, s>>>(stop); }

void launch_to_abi(const Launch &L, const double *x64, double *xabi, long long rhs0, long long nvalid) {
    const long long n = (long long)L.lat.N * L.nc * L.W;
    k_to_abi<<<blocks_for(n), kBlock, 0, L.stream>>>(L, (const double2 *)x64, (double2 *)xabi, rhs0, nvalid);
}

void launch_abi_to_internal(const Launch &L, int prec, const double *vabi, long long rhs0, long long nvalid,
                            void *out) {
    const long long n = (long long)L.lat.N * L.nc * L.W;
    DP_DISPATCH_PREC(prec, S,
                     k_abi_to_internal<S><<<blocks_for(n), kBlock, 0, L.stream>>>(L, (const double2 *)vabi, rhs0,
                                                                                  nvalid, (S *)out));
}

void launch_internal_to_abi_prec(const Launch &L, int prec, const void *in, double *yabi, long long rhs0,
                                 long long nvalid) {
    const long long n = (long long)L.lat.N * L.nc * L.W;
    DP_DISPATCH_PREC(prec, S,
                     k_internal_to_abi<S><<<blocks_for(n), kBlock, 0, L.stream>>>(L, (const S *)in, (double2 *)yabi,
                                                                                  rhs0, nvalid));
}

void launch_make_probes_abi(const Lat &lat, int nc, const ProbeGen &g, long long nrhs, double *out, hipStream_t s) {
    const long long n = nrhs * lat.N * nc;
    k_probes_abi<<<blocks_for(n), kBlock, 0, s>>>(lat, nc, g, nrhs, (double2 *)out);
}

// ------------------------------------------------------------ multi-instance launchers

template <typename S, int NC, bool LINKS, int M, int KIND>
static void b_stencil_m(const BatchLaunch &B, hipEvent_t ev0, hipEvent_t ev1) {
    if (ev0)
        hipExtLaunchKernelGGL(k_b_stencil<S, S, NC, LINKS, M, KIND>, dim3(B.nblocks), dim3(kBlock), 0, B.stream, ev0,
                              ev1, 0, B);
    else
        k_b_stencil<S, S, NC, LINKS, M, KIND><<<B.nblocks, kBlock, 0, B.stream>>>(B);
}

template <typename S, int NC, bool LINKS, int KIND>
static void b_stencil_t(const BatchLaunch &B, hipEvent_t ev0, hipEvent_t ev1) {
    if (B.mode == 1)
        b_stencil_m<S, NC, LINKS, 1, KIND>(B, ev0, ev1);
    else
        b_stencil_m<S, NC, LINKS, 0, KIND>(B, ev0, ev1);
}

template <int KIND>
static void b_stencil(const BatchLaunch &B, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr) {
    DP_DISPATCH_PREC(B.prec, S, {
        if (B.nc == 3)
            B.links ? b_stencil_t<S, 3, true, KIND>(B, ev0, ev1) : b_stencil_t<S, 3, false, KIND>(B, ev0, ev1);
        else
            B.links ? b_stencil_t<S, 1, true, KIND>(B, ev0, ev1) : b_stencil_t<S, 1, false, KIND>(B, ev0, ev1);
    });
}

template <typename S, int NC, bool LINKS>
static void b_init_probe_t(const BatchLaunch &B) {
    k_b_init_probe<S, NC, LINKS><<<B.nblocks, kBlock, 0, B.stream>>>(B);
}

void launch_b_init(const BatchLaunch &B) {
    if (B.eo) {
        DP_DISPATCH_PREC(B.prec, S, {
            if (B.nc == 3)
                B.links ? b_init_probe_t<S, 3, true>(B) : b_init_probe_t<S, 3, false>(B);
            else
                B.links ? b_init_probe_t<S, 1, true>(B) : b_init_probe_t<S, 1, false>(B);
        });
        k_b_finish<4, kEpiInitEo><<<B.nslots * B.W, kBlock, 0, B.stream>>>(B, kSlotInit);
    } else {
        DP_DISPATCH_PREC(B.prec, S, k_b_init<S><<<B.nblocks, kBlock, 0, B.stream>>>(B));
        k_b_finish<2, kEpiInit><<<B.nslots * B.W, kBlock, 0, B.stream>>>(B, kSlotInit);
    }
}

void launch_b_hop(const BatchLaunch &B, hipEvent_t ev0, hipEvent_t ev1) { b_stencil<kStHop>(B, ev0, ev1); }

void launch_b_stencil(const BatchLaunch &B, hipEvent_t ev0, hipEvent_t ev1) { b_stencil<kStFull>(B, ev0, ev1); }

template <typename S, int XNT>
static void b_update_t(const BatchLaunch &B, int xmode) {
    if constexpr (!std::is_same<S, double2>::value) {
        if (xmode == 1) return k_b_update<S, 1, XNT><<<B.nblocks, kBlock, 0, B.stream>>>(B);
        if (xmode == 2) return k_b_update<S, 2, XNT><<<B.nblocks, kBlock, 0, B.stream>>>(B);
    }
    k_b_update<S, 0, XNT><<<B.nblocks, kBlock, 0, B.stream>>>(B);
}

void launch_b_update(const BatchLaunch &B, int xmode) {
    // With few slots a slot has many workgroups, and a wavefront would add up
    // its lane's partials in many rounds (9 instances, 9216 workgroups: 10.2 us,
    // 5.7 with a workgroup per lane); with many slots there are few partials
    // and many lanes (256 slots of 64 workgroups: 12.8 us, and 26).
    if (B.nblocks / B.nslots > 128)
        k_b_finish_cg_wide<<<B.nslots * B.W, kBlock, 0, B.stream>>>(B);
    else
        k_b_finish_cg<<<(B.nslots * B.W + kBlock / 64 - 1) / (kBlock / 64), kBlock, 0, B.stream>>>(B);
    DP_DISPATCH_PREC(B.prec, S,
                     B.xnt == 0   ? b_update_t<S, 0>(B, xmode)
                     : B.xnt == 1 ? b_update_t<S, 1>(B, xmode)
                                  : b_update_t<S, 2>(B, xmode));
}

void launch_b_reseed(const BatchLaunch &B) { k_b_reseed<<<B.nslots * B.W, kBlock, 0, B.stream>>>(B); }

void launch_b_iteration(const BatchLaunch &B, int xmode) {
    if (B.eo) launch_b_hop(B);
    launch_b_stencil(B);
    launch_b_update(B, xmode);
}

template <typename S, int NC, bool LINKS>
static void b_tr_t(const BatchLaunch &B, int phase, int ru) {
    if (B.mode == 1)
        k_b_true_resid<S, NC, LINKS, 1><<<B.nblocks, kBlock, 0, B.stream>>>(B, phase, ru);
    else
        k_b_true_resid<S, NC, LINKS, 0><<<B.nblocks, kBlock, 0, B.stream>>>(B, phase, ru);
}

template <int NC, bool LINKS>
static void b_odd_x_t(const BatchLaunch &B, int phase) {
    if (B.mode == 1)
        k_b_odd_x<NC, LINKS, 1><<<B.nblocks, kBlock, 0, B.stream>>>(B, phase);
    else
        k_b_odd_x<NC, LINKS, 0><<<B.nblocks, kBlock, 0, B.stream>>>(B, phase);
}

static void b_odd_x(const BatchLaunch &B, int phase) {
    if (B.nc == 3)
        B.links ? b_odd_x_t<3, true>(B, phase) : b_odd_x_t<3, false>(B, phase);
    else
        B.links ? b_odd_x_t<1, true>(B, phase) : b_odd_x_t<1, false>(B, phase);
}

// Reliable update (final_stats = 0: slots flagged kSlotRU; mixed precision:
// fold, then the true residual replaces r and continues p) or the final
// statistics (final_stats = 1: slots flagged kSlotFinal; the true residual's norm
// only: FP64, whose iterate is already the solution, and mixed slots that no
// update has folded yet, having had no active lane).
void launch_b_ru(const BatchLaunch &B, int final_stats) {
    const int phase = final_stats ? kSlotFinal : kSlotRU;
    const int ru = final_stats ? 0 : 1;
    DP_DISPATCH_PREC(B.prec, S, {
        if (B.prec != kF64) k_b_fold<S><<<B.nblocks, kBlock, 0, B.stream>>>(B, phase);
        if (B.eo) b_odd_x(B, phase);
        if (B.nc == 3)
            B.links ? b_tr_t<S, 3, true>(B, phase, ru) : b_tr_t<S, 3, false>(B, phase, ru);
        else
            B.links ? b_tr_t<S, 1, true>(B, phase, ru) : b_tr_t<S, 1, false>(B, phase, ru);
    });
    if (final_stats)
        k_b_finish<2, kEpiStats><<<B.nslots * B.W, kBlock, 0, B.stream>>>(B, phase);
    else
        k_b_finish<2, kEpiRU><<<B.nslots * B.W, kBlock, 0, B.stream>>>(B, phase);
}

void launch_b_dot(const BatchLaunch &B) {
    k_b_dot<<<B.nblocks, kBlock, 0, B.stream>>>(B);
    k_b_finish<2, kEpiTj><<<B.nslots * B.W, kBlock, 0, B.stream>>>(B, kSlotFinal);
}

void launch_b_ctrl(const BatchLaunch &B) {
    k_b_finish<2, kEpiCheck><<<B.nslots * B.W, kBlock, 0, B.stream>>>(B, kSlotIter);
    k_b_ctrl<<<B.nslots, 64, 0, B.stream>>>(B);
}

void launch_b_count(const BatchLaunch &B) { k_b_ctrl<<<B.nslots, 64, 0, B.stream>>>(B); }

// Copies the CG state block of every slot flagged kSlotFinal (stride bytes,
// a multiple of 16) from st_all to dst, the device alias of a pinned host
// buffer with the same layout.
__global__ void k_b_state_out(BatchLaunch B, const char *__restrict__ st_all, char *__restrict__ dst, size_t stride) {
    const SlotDesc *d = B.sd + blockIdx.x;
    if (!(d->flags & kSlotFinal)) return;
    const uint4 *src = (const uint4 *)(st_all + stride * blockIdx.x);
    uint4 *out = (uint4 *)(dst + stride * blockIdx.x);
    for (size_t i = threadIdx.x; i < stride / 16; i += blockDim.x) out[i] = ldg(src + i);
}

// dst[0 .. bytes) = src[0 .. bytes): bytes a multiple of 4; src may be the
// device alias of pinned host memory
__global__ void k_copy_in(void *__restrict__ dst, const void *__restrict__ src, size_t bytes) {
    const size_t n16 = bytes / 16;
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x, st = (size_t)gridDim.x * blockDim.x;
    for (size_t i = i0; i < n16; i += st) stg((uint4 *)dst + i, ldg((const uint4 *)src + i));
    for (size_t i = n16 * 4 + i0; i < bytes / 4; i += st) stg((uint32_t *)dst + i, ldg((const uint32_t *)src + i));
}

void launch_copy_in(void *dst, const void *src, size_t bytes, hipStream_t s) {
    if (!bytes) return;
    const int blocks = (int)std::min<size_t>(64, (bytes / 16 + kBlock - 1) / kBlock + 1);
    k_copy_in<<<blocks, kBlock, 0, s>>>(dst, src, bytes);
}

void launch_b_state_out(const BatchLaunch &B, const char *st_all, char *dst, size_t stride) {
    k_b_state_out<<<B.nslots, kBlock, 0, B.stream>>>(B, st_all, dst, stride);
}


void launch_probe_fill(const Launch &L, const ProbeGen &g, double *out) {
    k_probe_fill<<<L.nblk, kBlock, 0, L.stream>>>(L, g, (double2 *)out);
}

void launch_init_b64(const Launch &L, int prec, const double *src, const InitArgs &ia) {
    init_block<2>(L, prec, ProbeGen{}, src, 0, 0, ia);
}

void launch_dot_shift(const Launch &L, const double *u, const double *w, int p, const Red &rd, const CgState &cs) {
    k_dot_shift<<<L.nblk, kBlock, 0, L.stream>>>(L, (const double2 *)u, (const double2 *)w, p, rd);
    k_finish<2, kEpiTj><<<L.W, kBlock, 0, L.stream>>>(rd, cs);
}

void launch_resid_norm(const Launch &L, const double *u, const double *w, const double *theta, const Red &rd,
                       const CgState &cs) {
    k_resid_norm<<<L.nblk, kBlock, 0, L.stream>>>(L, (const double2 *)u, (const double2 *)w, theta, rd);
    k_finish<1, kEpiStatsP1><<<L.W, kBlock, 0, L.stream>>>(rd, cs);
}

void launch_axpby(long long n, double a, const double *q, double b, const double *v, double *out, hipStream_t s) {
    k_axpby<<<blocks_for(n), kBlock, 0, s>>>(n, a, (const double2 *)q, b, (const double2 *)v, (double2 *)out);
}

void launch_rand_fill(long long n, unsigned long long seed, double *v, hipStream_t s) {
    k_rand_fill<<<blocks_for(n), kBlock, 0, s>>>(n, seed, (double2 *)v);
}

void launch_scale_lanes(long long n, int W, const double *sc, const double *v, double *out, hipStream_t s) {
    k_scale_lanes<<<blocks_for(n), kBlock, 0, s>>>(n, W, sc, (const double2 *)v, (double2 *)out);
}

int gram_row_blocks(long long n) { return (int)std::max<long long>(1, std::min<long long>(256, n / 512)); }

void launch_gram(long long n, int WX, int WY, const double *X, const double *Y, double *part, double scale, double *H,
                 hipStream_t s) {
    const int nrb = gram_row_blocks(n);
    const int tiles = ((WX + kGramTile - 1) / kGramTile) * ((WY + kGramTile - 1) / kGramTile);
    k_gram<<<dim3(nrb, tiles), kBlock, 0, s>>>(n, WX, WY, (const double2 *)X, (const double2 *)Y, (double2 *)part);
    k_gram_reduce<<<(WX * WY + 15) / 16, kBlock, 0, s>>>(nrb, WX, WY, (const double2 *)part, scale,
                                                                   (double2 *)H);
}

void launch_rot(long long n, int WX, int WY, const double *X, const double *C, double *out, int accumulate,
                hipStream_t s) {
    k_rot<<<blocks_for(n * WY), kBlock, 0, s>>>(n, WX, WY, (const double2 *)X, (const double2 *)C, (double2 *)out,
                                               accumulate);
}

void launch_hop_bound(const Lat &lat, int nc, const double *U8, double *out, hipStream_t s) {
    k_hop_bound<<<blocks_for(lat.N), kBlock, 0, s>>>(lat, nc, (const double2 *)U8, out);
}

}  // namespace dp

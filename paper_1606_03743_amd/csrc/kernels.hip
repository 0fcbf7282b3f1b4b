// HIP kernels for gfx950 (MI355X): Gaussian-cubature potential and field of charged
// BEM triangles and rectangles (Glueck & Hilk, arXiv:1606.03743).
//
//  near_list_kernel    FP64 distance-ratio test (Sec. 2) behind boxes of points; near pairs
//                      compacted per wavefront into a dense list.
//  far_eval_kernel     PPT field points per lane; element tiles are staged in LDS with
//                      their Gaussian points generated on the fly in each element's own
//                      frame (Eq. 3.2 / 3.3); the same test per pair leaves the near ones out;
//                      far pairs summed as point charges (Sec. 4, Eq. 4.1), potential and field
//                      from the same nodes.  FP64 or mixed (FP32 node sums); one rule per element
//                      kind or the rule chosen by distance ratio; potential and field, potential
//                      alone or field gradient.
//  far_few_kernel      the same for at most 128 points: an element per lane, FP64 sums, the near
//                      pairs listed in the same launch.
//  far_colloc_kernel   the same sum, potential only, at element centroids, for up to eight
//                      density vectors (matrix-free collocation product).
//  near_kernel         FP64 near field over the dense list: each pair's recursive subdivision
//                      (triangle: four midpoint children; rectangle: 2 x 2) is walked in lattice
//                      coordinates; a child at DR >= near_dr of its own (or at the depth cap) gets
//                      the element's rule.  Deep pairs, and all pairs of a short list, are walked
//                      breadth first by a wavefront each; the others one per lane depth first,
//                      64 leaves at a time taking the rule together.  Pairs are handed out the most
//                      expensive first (near_order.hip).  Each pair's result goes to its
//                      own slot in (point, element) order; the per-point sums are formed in
//                      that order afterwards (near_order.hip), so results are reproducible
//                      bit for bit.
//                      Pairs whose point lies on the element (found by the cost pass, last in
//                      the order) get the exact polar integral, one lane per pair, after the
//                      walk loop: kept out of the loop so that the depth-first walk's register
//                      footprint stays below 128 VGPRs, and its workgroups fit beside the far
//                      kernels of other streams.
#include "bemc_internal.h"
#include "on_element.h"

namespace bemc {

constexpr double kEps0 = 8.8541878188e-12;  // vacuum permittivity, CODATA 2022 (F/m)
double coulomb_constant() { return 1.0 / (4.0 * 3.14159265358979323846 * kEps0); }

namespace {

constexpr int kBlock = 256;       // 4 wavefronts
constexpr int kTileNodes = 1024;  // Gaussian-point slots of one LDS tile
constexpr int kMaxTileElems = 64;

// elements of one LDS tile for nn nodes an element
template <typename Lds>
__device__ __forceinline__ int tile_elems(int nn) { return min(Lds::kElems, max(1, Lds::kNodes / nn)); }

__device__ __forceinline__ float rsqrt32(float x) { return __builtin_amdgcn_rsqf(x); }

// Negative half powers in FP64, x^(-P/2) / kappa: with the hardware estimate y (~24 bits) and
// e = 1 - x y^2, x^(-P/2) = y^P (1 + P e/2 + P (P + 2) e^2 / 8 + O(e^3)) to full precision (the
// next term is below 1e-20).  Written as a square, the polynomial is kappa ((e + h)^2 + c) with
// h = 2 / (P + 2) and kappa = P (P + 2) / 8: two instructions instead of three, and the power
// y^P needs no refined 1/r first.  The constant kappa is left out here and multiplied into the
// element's charge once (half_power_scale).  kHalf = 1 + h and kRest = c are chosen among the
// neighbouring FP64 numbers so that kappa (h^2 + c) = 1 to 2e-17.  Relative error against
// 64-bit-mantissa references: r^-3 rms 9.6e-17, max 3.8e-16 (cubing a refined 1/r: 1.7e-16 and
// 5.8e-16); r^-1 as x times r^-3 rms 9.6e-17.
template <int P> struct HalfPower;
template <> struct HalfPower<1> { static constexpr double kHalf = 0x1.aaaaaaaaaaaacp+0, kRest = 0x1.1c71c71c71c71p+1, kappa = 0.375; };
template <> struct HalfPower<3> { static constexpr double kHalf = 0x1.6666666666666p+0, kRest = 0x1.7e4b17e4b17e6p-2, kappa = 1.875; };
template <> struct HalfPower<5> { static constexpr double kHalf = 0x1.4924924924926p+0, kRest = 0x1.2cee3c9aa517ap-3, kappa = 4.375; };

// The factors y^P and (e + h)^2 + c of x^(-P/2) / kappa for P = 3.
__device__ __forceinline__ void half_power3(double x, double& y3, double& m)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double y2 = y * y;
    const double t = fma(-x, y2, HalfPower<3>::kHalf);
    m = fma(t, t, HalfPower<3>::kRest);
    y3 = y2 * y;
}

// x^(-3/2) over half_power_scale<3, T>
__device__ __forceinline__ double inv_cube(double x)
{
    double y3, m;
    half_power3(x, y3, m);
    return y3 * m;
}
__device__ __forceinline__ float inv_cube(float x)
{
    const float y = rsqrt32(x);
    return (y * y) * y;
}

// w x^(-5/2) over half_power_scale<5, T>
__device__ __forceinline__ double inv_fifth(double w, double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double y2 = y * y;
    const double t = fma(-x, y2, HalfPower<5>::kHalf);
    const double m = fma(t, t, HalfPower<5>::kRest);
    return ((w * y) * (y2 * y2)) * m;
}
__device__ __forceinline__ float inv_fifth(float w, float x)
{
    const float y = rsqrt32(x);
    const float y2 = y * y;
    return (w * y) * (y2 * y2);
}

// acc + w x^(-1/2) / kappa in FP64 (w = 1: one instruction less)
__device__ __forceinline__ double add_inv_root(double x, double acc)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double t = fma(-(x * y), y, HalfPower<1>::kHalf);
    return fma(y, fma(t, t, HalfPower<1>::kRest), acc);
}
__device__ __forceinline__ double add_inv_root(double w, double x, double acc)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double t = fma(-(x * y), y, HalfPower<1>::kHalf);
    return fma(w * y, fma(t, t, HalfPower<1>::kRest), acc);
}

// kappa of the node sums that P and T stand for: FP64 sums lack it, FP32 sums do not
template <int P, typename T>
constexpr double half_power_scale() { return std::is_same<T, double>::value ? HalfPower<P>::kappa : 1.0; }

__device__ __forceinline__ int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }

// The lanes of the wavefront for which pred holds.  A comparison's own lane mask: __ballot
// takes an int, and turning the comparison into one and back costs two more vector
// instructions per call.
__device__ __forceinline__ unsigned long long lane_mask(bool pred) { return __builtin_amdgcn_ballot_w64(pred); }

// number of set bits of m below this lane
__device__ __forceinline__ unsigned lanes_below(unsigned long long m)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

__device__ __forceinline__ unsigned long long bcast_u64(unsigned long long v, int src)
{
    const unsigned lo = __shfl((unsigned)v, src);
    const unsigned hi = __shfl((unsigned)(v >> 32), src);
    return ((unsigned long long)hi << 32) | lo;
}

// v of one lane, the same in every lane (a scalar)
__device__ __forceinline__ double read_lane(double v, int lane)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = __builtin_amdgcn_readlane((unsigned)b, lane), hi = __builtin_amdgcn_readlane((unsigned)(b >> 32), lane);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// LDS written by some lanes of a wavefront, read by others: finish the writes first.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Near pairs of one wavefront on their way to the list: compacted into a buffer of its own in
// LDS (lane offsets by popcount), which goes to the list with one atomic on the list's length
// when another 64 pairs might not fit.  Appending each candidate's pairs with an atomic of its
// own bound the pass: they all hit one address (32,768 points x 150,000 elements, 697,000 pairs:
// see near_list_kernel).  Called with every lane of the wavefront active.
template <unsigned SIZE>
struct NearBuffer {
    NearPair* buf;  // [SIZE]
    unsigned n;     // pairs held (the same in every lane)

    __device__ __forceinline__ void flush(NearPair* list, unsigned long long cap, DevCounters* ctr)
    {
        if (n == 0) return;
        wave_lds_sync();
        unsigned long long base = 0;
        if (lane_id() == 0) base = atomicAdd(&ctr->near_count, (unsigned long long)n);
        base = bcast_u64(base, 0);
        for (unsigned i = lane_id(); i < n; i += 64)
            if (base + i < cap) list[base + i] = buf[i];
        wave_lds_sync();
        n = 0;
    }
    __device__ __forceinline__ void record(bool is_near, uint32_t p, uint32_t e, NearPair* list,
                                           unsigned long long cap, DevCounters* ctr)
    {
        const unsigned long long m = lane_mask(is_near);
        if (m == 0ull) return;
        if (is_near) buf[n + lanes_below(m)] = NearPair{ p, e };
        n += (unsigned)__popcll(m);
        if (n > SIZE - 64) flush(list, cap, ctr);
    }
};

// Near pairs straight to the list, one atomic per wavefront that has any (few points: a few
// wavefronts of a launch do).  Called with every lane of the wavefront active.
__device__ __forceinline__ void append_near(bool is_near, uint32_t p, uint32_t e, NearPair* list,
                                            unsigned long long cap, DevCounters* ctr)
{
    const unsigned long long m = lane_mask(is_near);
    if (m == 0ull) return;
    unsigned long long base = 0;
    if (lane_id() == 0) base = atomicAdd(&ctr->near_count, (unsigned long long)__popcll(m));
    base = bcast_u64(base, 0) + lanes_below(m);
    if (is_near && base < cap) list[base] = NearPair{ p, e };
}

// ------------------------------------------------------------- near-pair list -----
// An axis-aligned box: low and high corner.
struct Box {
    double lo[3], hi[3];

    // is a centroid within its threshold t2 = (near_dr L)^2 of the box?  (an empty box: no)
    __device__ __forceinline__ bool in_reach(double cx, double cy, double cz, double t2) const
    {
        const double dx = fmax(fmax(lo[0] - cx, cx - hi[0]), 0.0);
        const double dy = fmax(fmax(lo[1] - cy, cy - hi[1]), 0.0);
        const double dz = fmax(fmax(lo[2] - cz, cz - hi[2]), 0.0);
        return fma(dx, dx, fma(dy, dy, dz * dz)) < t2;
    }
};

// One axis of split_boxes: the least and greatest of the lanes up to this one (pl, ph) and of the
// later ones (sl, sh).
__device__ __forceinline__ void split_axis(double lo, double hi, double& pl, double& ph, double& sl, double& sh)
{
    const int lane = lane_id();
    pl = sl = lo;
    ph = sh = hi;
    for (int o = 1; o < 64; o <<= 1) {
        const double a = __shfl_up(pl, o), b = __shfl_up(ph, o), c = __shfl_down(sl, o), d = __shfl_down(sh, o);
        if (lane >= o) { pl = fmin(pl, a); ph = fmax(ph, b); }
        if (lane + o < 64) { sl = fmin(sl, c); sh = fmax(sh, d); }
    }
    sl = __shfl_down(sl, 1);
    sh = __shfl_down(sh, 1);
    if (lane == 63) { sl = INFINITY; sh = -INFINITY; }
}

// Two boxes for the wavefront's points (one per lane; an invalid lane's is empty): the points up
// to a lane and those after it, where their edges add up to least.  (The axes are scanned twice,
// one at a time: keeping all three takes 60 registers more.)
__device__ __forceinline__ void split_boxes(const Box& own, Box& a, Box& b)
{
    double cost = 0.0, pl, ph, sl, sh;
#pragma unroll 1
    for (int c = 0; c < 3; ++c) {
        const double lo = c == 0 ? own.lo[0] : (c == 1 ? own.lo[1] : own.lo[2]);
        const double hi = c == 0 ? own.hi[0] : (c == 1 ? own.hi[1] : own.hi[2]);
        split_axis(lo, hi, pl, ph, sl, sh);
        cost += fmax(ph - pl, 0.0) + fmax(sh - sl, 0.0);
    }
    double least = cost;
    for (int o = 32; o > 0; o >>= 1) least = fmin(least, __shfl_xor(least, o));
    const unsigned long long at = lane_mask(cost == least);
    const int split = at ? (int)__builtin_ctzll(at) : 63;  // (no lane: coordinates that are not numbers)
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        split_axis(own.lo[c], own.hi[c], pl, ph, sl, sh);
        a.lo[c] = read_lane(pl, split);  // (scalar registers: the boxes stay live to the end)
        a.hi[c] = read_lane(ph, split);
        b.lo[c] = read_lane(sl, split);
        b.hi[c] = read_lane(sh, split);
    }
}

// Every (point, element) pair with D^2 < (near_dr L)^2 (the distance-ratio switch, Sec. 2)
// goes into the near-pair list, compacted per wavefront (NearBuffer); pairs past the capacity are
// counted, not stored.  A workgroup takes kListPoints consecutive points (Morton order:
// neighbours in space) and one chunk of the elements (more chunks when the points are few),
// and bounds the points by a box; the elements whose centroid lies within near_dr L of that box
// are its candidates, kept in LDS, and 64 consecutive points take the per-point test of a candidate
// only when it passes the same test with their own boxes (64 candidates at a time, one per lane).
// There are two boxes for them: a run of points across a step of the Morton curve spans the
// whole geometry, and the few such runs set the pass's time; split where the two parts' boxes
// are smallest, both are small.  With the buffered appends: 131,071 points x 150,000 elements
// 6.2 -> 0.57 ms (2.3 with one box), 32,768 points 3.0 -> 0.43 ms; 777 points x 3,600 elements 220 ->
// 23 us; 50,000 centroids 4.3 -> 0.42 ms.  Collocation: the points are the centroids
// themselves (the same [3][n] layout).
constexpr int kListPPT = 2;
constexpr int kListPoints = kBlock * kListPPT;
constexpr int64_t kListFine = 1024;  // elements of a chunk from which the points' own boxes pay

// FINE: with the points' own boxes, for long chunks (a short chunk's candidates are tested at once:
// forming the boxes takes longer, 30 us).  87 registers and 56 bytes of scratch per lane, 62 and none
// without the boxes, which is what fits beside four workgroups of another stream's mixed far kernel.
// Served batches take either by the same rule (1,000,000 elements: FINE above 1,024 points); without
// FINE there the latencies stay the same (40 queries/s by distance ratio: p50 36.6 and 35.7 ms, short queries
// 25.3 and 24.3, p99 537 and 541).
template <bool FINE>
__global__ __launch_bounds__(kBlock) void near_list_kernel(const double* __restrict__ pts, int64_t n, Elements el,
                                                           NearPair* __restrict__ list, unsigned long long cap,
                                                           DevCounters* __restrict__ ctr, int64_t chunk)
{
    __shared__ double wbox[kBlock / 64][6];
    __shared__ double box[6];
    __shared__ uint32_t cand[kBlock];
    __shared__ double4 cand_c[kBlock];  // the candidates' centroids and thresholds
    __shared__ int ncand;
    constexpr unsigned kListBuf = FINE ? 512 : 256;
    __shared__ NearPair pairs[kBlock / 64][kListBuf];
    const int64_t ne = el.ne;
    double x[kListPPT], y[kListPPT], z[kListPPT];
    bool valid[kListPPT];
    uint32_t idx[kListPPT];
    double lo[3] = { INFINITY, INFINITY, INFINITY }, hi[3] = { -INFINITY, -INFINITY, -INFINITY };
    Box part[kListPPT][2];
#pragma unroll
    for (int k = 0; k < kListPPT; ++k) {
        const int64_t p = (int64_t)blockIdx.x * kListPoints + (threadIdx.x / 64) * (64 * kListPPT) + k * 64 + lane_id();
        valid[k] = p < n;
        idx[k] = (uint32_t)p;
        x[k] = valid[k] ? pts[p] : 0.0;
        y[k] = valid[k] ? pts[n + p] : 0.0;
        z[k] = valid[k] ? pts[2 * n + p] : 0.0;
        if (valid[k]) {
            lo[0] = fmin(lo[0], x[k]); lo[1] = fmin(lo[1], y[k]); lo[2] = fmin(lo[2], z[k]);
            hi[0] = fmax(hi[0], x[k]); hi[1] = fmax(hi[1], y[k]); hi[2] = fmax(hi[2], z[k]);
        }
        if constexpr (FINE) {
            const double e0 = valid[k] ? 0.0 : INFINITY;
            split_boxes(Box{ { x[k] + e0, y[k] + e0, z[k] + e0 }, { x[k] - e0, y[k] - e0, z[k] - e0 } }, part[k][0],
                        part[k][1]);
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
        for (int o = 32; o > 0; o >>= 1) {
            lo[c] = fmin(lo[c], __shfl_xor(lo[c], o));
            hi[c] = fmax(hi[c], __shfl_xor(hi[c], o));
        }
    const int wave = threadIdx.x / 64;
    if (lane_id() == 0) {
#pragma unroll
        for (int c = 0; c < 3; ++c) { wbox[wave][c] = lo[c]; wbox[wave][3 + c] = hi[c]; }
    }
    if (threadIdx.x == 0) ncand = 0;
    __syncthreads();
    if (threadIdx.x < 6) {
        double v = wbox[0][threadIdx.x];
        for (int w = 1; w < kBlock / 64; ++w) v = threadIdx.x < 3 ? fmin(v, wbox[w][threadIdx.x]) : fmax(v, wbox[w][threadIdx.x]);
        box[threadIdx.x] = v;
    }
    __syncthreads();
    NearBuffer<kListBuf> near{ pairs[wave], 0u };
    const Box all{ { box[0], box[1], box[2] }, { box[3], box[4], box[5] } };
    // this workgroup's chunk of the elements (blockIdx.y)
    const int64_t e_begin = (int64_t)blockIdx.y * chunk, e_end = min(ne, e_begin + chunk);
    for (int64_t c0 = e_begin; c0 < e_end; c0 += kBlock) {
        const int64_t e = c0 + threadIdx.x;
        bool hit = false;
        double cx = 0.0, cy = 0.0, cz = 0.0, t2 = 0.0;
        if (e < e_end) {
            cx = el.cen[e]; cy = el.cen[ne + e]; cz = el.cen[2 * ne + e]; t2 = el.thr2[e];
            hit = all.in_reach(cx, cy, cz, t2);
        }
        const unsigned long long m = lane_mask(hit);
        if (m) {
            int base = 0;
            if (lane_id() == 0) base = atomicAdd(&ncand, __popcll(m));
            base = __shfl(base, 0);
            if (hit) {
                cand[base + (int)lanes_below(m)] = (uint32_t)e;
                cand_c[base + (int)lanes_below(m)] = make_double4(cx, cy, cz, t2);
            }
        }
        __syncthreads();
        const int nc = ncand;
        for (int i0 = 0; i0 < nc; i0 += 64) {
            bool mine[kListPPT] = {};
            if (i0 + lane_id() < nc) {
                const double4 cc = cand_c[i0 + lane_id()];
#pragma unroll
                for (int k = 0; k < kListPPT; ++k)
                    mine[k] = !FINE || part[k][0].in_reach(cc.x, cc.y, cc.z, cc.w) || part[k][1].in_reach(cc.x, cc.y, cc.z, cc.w);
            }
#pragma unroll
            for (int k = 0; k < kListPPT; ++k)
                for (unsigned long long todo = lane_mask(mine[k]); todo; todo &= todo - 1) {
                    const int i = i0 + __ffsll((long long)todo) - 1;
                    const double4 cc = cand_c[i];  // one LDS read for the whole wavefront
                    const double dx = x[k] - cc.x, dy = y[k] - cc.y, dz = z[k] - cc.z;
                    const bool nr = valid[k] && fma(dx, dx, fma(dy, dy, dz * dz)) < cc.w;
                    near.record(nr, idx[k], cand[i], list, cap, ctr);
                }
        }
        __syncthreads();
        if (threadIdx.x == 0) ncand = 0;
        __syncthreads();
    }
    near.flush(list, cap, ctr);
}

// ---------------------------------------------------------------- LDS staging ------
// Each element is summed in its own orthonormal frame: origin at the centroid, f1 and f2
// in its plane, f3 its unit normal.  A Gaussian point has in-plane coordinates (a, b).
//
// Expanded form (triangles, Table B rectangles, the short distance-ratio levels): with
// d = P - centroid, |p|^2 = D^2 from the distance test and q1 = -2 f1.d, q2 = -2 f2.d,
//   r^2 = D^2 + (a^2 + b^2) + q1 a + q2 b,
// and the field follows from the node sums S3 = sum w/r^3, S1 = sum w a/r^3, S2 = sum w b/r^3
// as E = q (S3 d - f1 S1 - f2 S2), rotated once per pair.  When every weight is positive,
// the nodes are staged divided by w^2, (a, b, a^2 + b^2, 1) / w^2: the reciprocal square
// root of r^2 / w^2 is w/r itself, and (w/r)^3 times the staged values gives the three
// field sums, which saves the multiplication by the weight per node.
//
// Rows form (the field of the 7 x 7 Gauss-Legendre rectangle rule): the point is
// rotated into the frame, p = (f1.d, f2.d, f3.d).  For rectangles f1 runs along the second
// side, so the nodes of a tensor Gauss-Legendre rule that share their first coordinate share
// b, and are summed in rows (pair_row).  The local field (sum w (p1 - a)/r^3, sum w (p2 - b)/r^3,
// p3 sum w/r^3) is rotated back with the frame.
enum FrameForm { kFrExp = 0, kFrRows = 1 };

// SMALL: half the nodes and elements (24 KB in FP64 instead of 47), for launches of one point per lane,
// whose registers would allow four workgroups a CU.
template <bool MIXED, int NRHS, bool SMALL>
struct TileLds {
    static constexpr int kNodes = SMALL ? kTileNodes / 2 : kTileNodes, kElems = SMALL ? kMaxTileElems / 2 : kMaxTileElems;
    using T = typename std::conditional<MIXED, float, double>::type;
    using T4 = typename std::conditional<MIXED, float4, double4>::type;
    T4 nd[kNodes];  // (a, b, a^2 + b^2, w), or divided by w^2 as (a, b, a^2 + b^2, 1) / w^2
    double cx[kElems], cy[kElems], cz[kElems], thr2[kElems];
    T fr[9][kElems];      // point rotation: expanded -2 f1, -2 f2 (gradient: f1, f2); rows f1, f2, f3
    double qr[9][kElems]; // rotation back scaled by the charge: expanded -q f1, -q f2;
                                 // rows q f1, q f2, q f3
    double q[NRHS][kElems];
    T lc[6][kElems];      // triangles: in-plane coordinates of A, B, C relative to the centroid
};

// Orbit structure of the compiled triangle rules (Tables A2-A5 as expanded on the host:
// the centroid first, then the S21 orbits with the distinct coordinate at A, B, C in turn,
// then the other orbits in groups of gs nodes).  A node of an S21 orbit lies on the line
// from the centroid to its vertex, at n = (l_k - l_other) u_k with u_k the vertex relative
// to the centroid, so d.n = s d.u_k needs one product per node once d.u_k is known per pair.
template <int NN> struct TriOrbits { static constexpr int nc = 0, n21 = 0, gs = 4; };
template <> struct TriOrbits<7> { static constexpr int nc = 1, n21 = 2, gs = 1; };    // Table A2
template <> struct TriOrbits<12> { static constexpr int nc = 0, n21 = 0, gs = 3; };   // Table A3 (cyclic)
template <> struct TriOrbits<19> { static constexpr int nc = 1, n21 = 4, gs = 6; };   // Table A4
template <> struct TriOrbits<33> { static constexpr int nc = 0, n21 = 5, gs = 6; };   // Table A5

// Staging form of the triangle nodes: levels back to back (one for a fixed rule), each with
// nc centroid nodes and n21 S21 nodes (three per orbit) in front.
struct TriForms {
    int nlev;
    int off[5];
    int nc[4], n21[4];
};

template <int NN, bool ORBITS>
__device__ __forceinline__ TriForms fixed_forms(int nn)
{
    TriForms t{ 1, { 0, nn, nn, nn, nn }, { 0, 0, 0, 0 }, { 0, 0, 0, 0 } };
    if (ORBITS) {
        t.nc[0] = TriOrbits<NN>::nc;
        t.n21[0] = 3 * TriOrbits<NN>::n21;
    }
    return t;
}

// Pair rows of the 7 x 7 Gauss-Legendre rectangle rule (node i*7 + j at natural coordinates
// (x_i, x_j)): the row of x_i has b = x_i beta and the nodes a = a0 + x_j alpha, a0 = x_i gamma,
// with x_{6-j} = -x_j, the same weight for j and 6 - j and x_3 = 0.  Four slots per row:
//   header (b, a0, w of the middle node, a0^2 + b^2), then per pair j = 0, 1, 2 with
//   s = x_{6-j} alpha: (s, s^2, w, w s).
// Folded (FP64 field and potential): 1 / w^2 in place of w in the header, and per pair (s, s^2, 1, 0) / w^2.
constexpr int kPairRowSlots = 28;
template <bool FOLDED>
__device__ __forceinline__ double4 pair_row_slot(const RuleTables& R, int prow, int m, double gamma, double beta,
                                                 double alpha)
{
    const int r = m >> 2, c = m & 3;
    if (c == 0) {
        const int i = prow + r * 7 + 3;
        const double x = R.rect[4 * i];
        const double b = x * beta, a0 = x * gamma;
        return make_double4(b, a0, FOLDED ? R.rect[4 * R.nr + i] : R.rect[4 * i + 2], fma(a0, a0, b * b));
    }
    const int i = prow + r * 7 + 7 - c;  // j = 6 - (c - 1)
    const double sv = R.rect[4 * i + 1] * alpha, w = R.rect[4 * i + 2];
    if constexpr (FOLDED) {
        const double iw2 = R.rect[4 * R.nr + i];
        return make_double4(sv * iw2, sv * sv * iw2, iw2, 0.0);
    }
    return make_double4(sv, sv * sv, w, w * sv);
}

// Gaussian points of elements [t0, t0 + te) in their frames (Eq. 3.2 / 3.3): triangle
// (a, b) = la A' + lb B' + lc C' from the in-plane coordinates of the vertices relative to
// the centroid; rectangle a = x gamma + y alpha, b = x beta for the rule point (x, y) in
// [-1, 1]^2 (alpha = |e2| / 2; beta, gamma the components of e1 / 2 across and along e2).
// FP32 tiles hold the FP64 values rounded once.  QR: stage the rotation back (field only).
// The first nfold nodes of each element are staged divided by w^2 (positive weights only).
// Nodes from prow on are a 7 x 7 Gauss-Legendre rule staged as pair rows (pair_row_slot).
// Triangles: centroid and S21 nodes (TriForms, folded nodes only) are staged as
// (0, 0, 1/w^2, 0) and (s, |n|^2, 1, 0) / w^2 with n = s u_k.  The charges are staged times
// scale (the constant that the node sums leave out, half_power_scale).
// GRAD (the gradient's sums): nothing is folded; the first nfold nodes are those of a rule whose
// orbits are known, the centroid and S21 nodes staged as (0, 0, 0, w) and (s, |n|^2, s^2, w).
template <bool TRI, bool MIXED, int FR, bool QR, bool GRAD, typename Lds>
__device__ __forceinline__ void stage_tile(Lds& s, const Elements& el, const RuleTables& R, int nn,
                                           int64_t t0, int te, int rhs0, int nrhs, int nfold, int prow,
                                           const TriForms& tf, double scale)
{
    using T = typename Lds::T;
    const int64_t ne = el.ne;
    // as many threads to an element as the workgroup has for a full tile (a power of two): each loads the
    // element's in-plane coordinates once and forms every per-th node (a thread per node loaded them
    // for each one and divided to find its element: with the levels' 71 and 85 nodes staging was a
    // tenth of the kernel; 131,071 points x 150,000 elements, mixed, potential: with the levels'
    // common case below 53.0 -> 46.9 ms, FP64 field of 100,000 107 -> 100 ms)
    const int lg = 31 - __builtin_clz((unsigned)(kBlock / tile_elems<Lds>(nn))), per = 1 << lg;
    const int j = threadIdx.x >> lg, sub = threadIdx.x & (per - 1);
    if (j >= te) return;
    const int64_t e = t0 + j;
    const double q = QR ? scale * el.q[(int64_t)rhs0 * ne + e] : 0.0;
    if (sub == 0) {
        s.cx[j] = el.cen[e];
        s.cy[j] = el.cen[ne + e];
        s.cz[j] = el.cen[2 * ne + e];
        s.thr2[j] = el.thr2[e];
    }
    for (int r = sub; r < nrhs; r += per) s.q[r][j] = scale * el.q[(int64_t)(rhs0 + r) * ne + e];
    for (int c = sub; c < (FR == kFrExp ? 6 : 9); c += per) {
        const double f = el.frame[(int64_t)c * ne + e];
        s.fr[c][j] = (T)(FR == kFrExp && !GRAD ? -2.0 * f : f);
        if (QR) s.qr[c][j] = FR == kFrExp ? -q * f : q * f;
    }
    double lo[6];  // triangle: vertices in the frame; rectangle: gamma, beta, alpha
#pragma unroll
    for (int c = 0; c < (TRI ? 6 : 3); ++c) lo[c] = el.loc[(int64_t)c * ne + e];
    if (TRI && sub == per - 1) {
#pragma unroll
        for (int c = 0; c < 6; ++c) s.lc[c][j] = (T)lo[c];
    }
    auto put = [&](int i, double x, double y, double z, double w) {
        if constexpr (MIXED) s.nd[j * nn + i] = make_float4((float)x, (float)y, (float)z, (float)w);
        else s.nd[j * nn + i] = make_double4(x, y, z, w);
    };
    for (int i = sub; i < nn; i += per) {
        if (!TRI && i >= prow) {
            if (i - prow < kPairRowSlots) {
                const double4 v = pair_row_slot<!MIXED && !GRAD>(R, prow, i - prow, lo[0], lo[1], lo[2]);
                put(i, v.x, v.y, v.z, v.w);
            }
            continue;
        }
        const double* node = (TRI ? R.tri : R.rect) + 4 * i;
        const double iw2 = GRAD ? 1.0 : (TRI ? R.tri[4 * R.nt + i] : R.rect[4 * R.nr + i]);
        double a, b, w;
        if (TRI) {
            const double la = node[0], lb = node[1], lc = node[2];
            w = node[3];
            if (i < nfold) {
                // the level of node i (selects, not indexing: the forms stay in registers)
                int off_l = tf.off[0], nc_l = tf.nc[0], n21_l = tf.n21[0];
#pragma unroll
                for (int l = 1; l < 4; ++l)
                    if (l < tf.nlev && i >= tf.off[l]) { off_l = tf.off[l]; nc_l = tf.nc[l]; n21_l = tf.n21[l]; }
                const int il = i - off_l;
                if (il < nc_l + n21_l) {
                    double v0 = 0.0, v1 = 0.0;
                    if (il >= nc_l) {  // S21: the distinct coordinate at vertex kk
                        const int kk = (il - nc_l) % 3;
                        const double lk = kk == 0 ? la : (kk == 1 ? lb : lc);
                        const double lk1 = kk == 0 ? lb : (kk == 1 ? lc : la);
                        const double sv = lk - lk1;
                        const double na = sv * (kk == 0 ? lo[0] : (kk == 1 ? lo[2] : lo[4]));
                        const double nb = sv * (kk == 0 ? lo[1] : (kk == 1 ? lo[3] : lo[5]));
                        v0 = sv * iw2;
                        v1 = fma(na, na, nb * nb) * iw2;
                    }
                    put(i, v0, v1, GRAD ? v0 * v0 : iw2, GRAD ? w : 0.0);
                    continue;
                }
            }
            a = la * lo[0] + lb * lo[2] + lc * lo[4];
            b = la * lo[1] + lb * lo[3] + lc * lo[5];
        } else {
            w = node[2];
            a = node[0] * lo[0] + node[1] * lo[2];
            b = node[0] * lo[1];
        }
        double g = fma(a, a, b * b);
        if (!GRAD && i < nfold) {
            a *= iw2;
            b *= iw2;
            g *= iw2;
            w = iw2;
        }
        put(i, a, b, g, w);
    }
}

// ------------------------------------------------------------ far field: sums -------
// kFarField: per point phi, Ex, Ey, Ez.  kFarGrad: the field gradient dE_i/dx_j as xx, yy,
// zz, xy, xz, yz (each point charge contributes q (delta_ij r^2 - 3 d_i d_j) / r^5).
// kFarPhi: the potential only (collocation).
enum FarMode { kFarField = 0, kFarGrad = 1, kFarPhi = 2 };

template <int MODE>
struct Sums {
    static constexpr int kOut = MODE == kFarGrad ? 6 : (MODE == kFarField ? 4 : 1);   // outputs per point
    static constexpr int kNode = MODE == kFarGrad ? 6 : (MODE == kFarField ? 4 : 1);  // element sums per point
};

// The constant left out of the node sums, multiplied into the staged charges (half_power_scale).
template <int MODE, typename T>
constexpr double sum_scale()
{
    return MODE == kFarGrad ? half_power_scale<5, T>()
                            : (MODE == kFarField ? half_power_scale<3, T>() : half_power_scale<1, T>());
}

// Field points of one lane and their FP64 accumulators.
template <int PPT, int MODE>
struct PointSet {
    double x[PPT], y[PPT], z[PPT];
    bool valid[PPT];
    uint32_t idx[PPT];
    double acc[Sums<MODE>::kOut][PPT];
};

// The lane's points relative to the element in hand.
template <int PPT, typename T>
struct Local {
    T q1[PPT], q2[PPT], H[PPT];           // expanded: -2 f1.d, -2 f2.d, D^2
    T p1[PPT], p2[PPT], p3[PPT];          // rows: f1.d, f2.d, f3.d
    T ri0[PPT], t[PPT];                   // FP32 gradient: 1/D and 1/D^2 (q1, q2 are times 1/D^2)
    double dx[PPT], dy[PPT], dz[PPT];     // d = P - centroid (FP64)
};

// Runs term(i) for the nodes i = 1 .. n-1 of one element (node 0 is peeled off by the
// caller, so that the sums start from its terms instead of from zero).  Long rules (and
// run-time counts) go in groups of four with a separate remainder: this keeps the
// accumulators in place, where an unrolled loop with a remainder makes the compiler copy
// them every iteration.  The short rules of the distance-ratio levels use a plain
// unrolled loop.
template <int NN, typename Term>
__device__ __forceinline__ void for_nodes(int n, Term term)
{
    if (NN > 0 && NN < 32) {
#pragma unroll 4
        for (int i = 1; i < n; ++i) term(i);
        return;
    }
    int i = 1;
#pragma unroll 1
    for (; i + 4 <= n; i += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) term(i + u);
    }
    for (; i < n; ++i) term(i);
}

// One folded node of the field (r^2 / w^2 = x): returns (w/r)^3 and adds w/r to phi.  FP64: both
// from x^(-3/2) alone, since (w/r)^3 x = w/r: 13 FP64 instructions per expanded node instead of
// 15 with a refined 1/r (one of them the quarter-rate v_rsq_f64).
__device__ __forceinline__ double inv_cube_phi(double x, double& phi)
{
    const double w3 = inv_cube(x);
    phi = fma(w3, x, phi);
    return w3;
}
__device__ __forceinline__ float inv_cube_phi(float x, float& phi)
{
    const float wr = rsqrt32(x);
    phi += wr;
    return (wr * wr) * wr;
}
// The same for an unfolded node of weight w (r^2 = x): returns w/r^3 and adds w/r to phi.
__device__ __forceinline__ double inv_cube_phi(double w, double x, double& phi)
{
    double y3, m;
    half_power3(x, y3, m);
    const double w3 = (w * y3) * m;
    phi = fma(w3, x, phi);
    return w3;
}
__device__ __forceinline__ float inv_cube_phi(float w, float x, float& phi)
{
    const float ri = rsqrt32(x);
    const float wr = w * ri;
    phi += wr;
    return wr * (ri * ri);
}

// Node sums of one element per field point (unit element charge, Eq. 4.1; FP64 sums lack the
// factor half_power_scale), accumulated into
// o, whose sums start at -0.0 (so that adding the first node folds into an assignment).
//   kFarField, expanded: (sum w/r, sum w a/r^3, sum w b/r^3, sum w/r^3);
//              FOLD: the staged node is (a, b, g, 1) / w^2 and rsqrt(r^2 / w^2) = w/r;
//   kFarPhi,   expanded: sum w/r;
//   kFarGrad,  unfolded: (S5 = sum w/r^5, Sa = sum w a/r^5, Sb = sum w b/r^5, sum w a^2/r^5,
//              sum w a b/r^5, sum w (a^2 + b^2)/r^5), from which add_element forms the tensor and
//              sum w/r^3 once per pair: 17 instructions per node beside the reciprocal
//              square root, 22 with the node's own offsets and both powers (far kernel, 15,000
//              points x 150,000 elements, 33-point / 7 x 7, FP64: 73.0 -> 53.9 ms; mixed, 50,001 x
//              18,000: 17.8 -> 11.9 ms).  FP32: r^2 is taken
//              over D^2 (grad_base), so that no power of a length above the square appears in
//              single precision: sizes down to 1e-18 and up to 1e18 of the geometry's unit.
template <int PPT, typename T>
__device__ __forceinline__ T grad_base(const Local<PPT, T>& L, int k, T g)  // D^2 + g, or over D^2
{
    if constexpr (std::is_same<T, double>::value) return L.H[k] + g;
    else return fma(L.t[k], g, T(1));
}
template <int PPT, int MODE, bool FOLD, typename T, typename T4>
__device__ __forceinline__ void node_term(const T4 Q, const Local<PPT, T>& L, T (&o)[Sums<MODE>::kNode][PPT])
{
    constexpr bool F64 = std::is_same<T, double>::value;
    const T a = Q.x, b = Q.y, g = Q.z, w = Q.w;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        if constexpr (MODE == kFarGrad) {
            const T w5 = inv_fifth(w, fma(L.q1[k], a, fma(L.q2[k], b, grad_base(L, k, g))));
            const T ua = w5 * a;
            o[0][k] += w5;
            o[1][k] += ua;
            o[2][k] = fma(w5, b, o[2][k]);
            o[3][k] = fma(ua, a, o[3][k]);
            o[4][k] = fma(ua, b, o[4][k]);
            o[5][k] = fma(w5, g, o[5][k]);
        } else if constexpr (FOLD) {
            const T x = fma(L.q1[k], a, fma(L.q2[k], b, fma(L.H[k], w, g)));  // r^2 / w^2
            if constexpr (MODE == kFarPhi) {
                if constexpr (F64) o[0][k] = add_inv_root(x, o[0][k]);
                else o[0][k] += rsqrt32(x);
            } else {
                const T wr3 = inv_cube_phi(x, o[0][k]);
                o[1][k] = fma(wr3, a, o[1][k]);
                o[2][k] = fma(wr3, b, o[2][k]);
                o[3][k] = fma(wr3, w, o[3][k]);
            }
        } else {
            const T x = fma(L.q1[k], a, fma(L.q2[k], b, L.H[k] + g));
            if constexpr (MODE == kFarPhi) {
                if constexpr (F64) o[0][k] = add_inv_root(w, x, o[0][k]);
                else o[0][k] = fma(w, rsqrt32(x), o[0][k]);
            } else {
                const T w3 = inv_cube_phi(w, x, o[0][k]);
                o[1][k] = fma(w3, a, o[1][k]);
                o[2][k] = fma(w3, b, o[2][k]);
                o[3][k] += w3;
            }
        }
    }
}

// One pair row of the 7 x 7 rule (slots n0 .. n0 + 3, see pair_row_slot) for potential and
// field, or the potential alone.  With da0 = p1 - a0 and C = |d - (a0 f1 + b f2)|^2, formed
// like the expanded form from D^2 (C = D^2 + a0^2 + b^2 - 2 (p1 a0 + p2 b): the rotation's
// rounding then enters only through the small products), the pair at a0 -+ s has
// r^2 = C + s^2 -+ 2 da0 s.  Per row the field's local parts follow from sg, the sum over the row
// of w/r^3, as E1 += da0 sg, E2 += (p2 - b) sg, S3 += sg; E1 -= SA once per element, SA the sum
// of w s (1/r+^3 - 1/r-^3).
// FP64 (folded slots): the potential comes from the same sums, since w/r = (w/r^3) r^2: over the
// row C sg - 2 da0 sa + sum w s^2 (1/r+^3 + 1/r-^3), sa the row's share of SA; the first term is
// close to the whole and the others small corrections, so nothing cancels.  9 FP64 instructions
// per node beside the reciprocal square root, 11.5 with refined 1/r and separate potential sums.
// FP32: 1/r is at hand, and the potential sums it: w (1/r+ + 1/r-).
template <int PPT, int MODE, typename T, typename T4>
__device__ __forceinline__ void pair_row(const T4* t, int n0, const Local<PPT, T>& L, T (&o)[Sums<MODE>::kNode][PPT],
                                         T (&SA)[PPT])
{
    constexpr bool F64 = std::is_same<T, double>::value;
    const T4 hd = t[n0];
    const T b = hd.x, a0 = hd.y, wc = hd.z, g0 = hd.w;
    T db[PPT], da0[PPT], C[PPT], mq[PPT], sg[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        C[k] = fma(L.q1[k], a0, fma(L.q2[k], b, L.H[k] + g0));
        if constexpr (MODE == kFarPhi) {
            mq[k] = fma(T(2), a0, L.q1[k]);
        } else {
            db[k] = L.p2[k] - b;
            da0[k] = L.p1[k] - a0;
            mq[k] = T(-2) * da0[k];
        }
    }
    // the middle node (a = a0)
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        if constexpr (MODE == kFarPhi) {
            if constexpr (F64) o[0][k] = add_inv_root(C[k] * wc, o[0][k]);
            else o[0][k] = fma(wc, rsqrt32(C[k]), o[0][k]);
        } else if constexpr (F64) {
            sg[k] = inv_cube(C[k] * wc) * wc;
        } else {
            const T ri = rsqrt32(C[k]);
            o[0][k] = fma(wc, ri, o[0][k]);
            sg[k] = wc * ((ri * ri) * ri);
        }
    }
    T sa[PPT];  // FP64 field: the row's sum w s (1/r+^3 - 1/r-^3)
#pragma unroll
    for (int pi = 1; pi <= 3; ++pi) {
        const T4 Q = t[n0 + pi];
        const T sv = Q.x, s2 = Q.y, w = Q.z, ws = Q.w;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            if constexpr (F64) {
                const T u = fma(C[k], w, s2);  // (C + s^2) / w^2
                const T xp = fma(mq[k], sv, u), xm = fma(-mq[k], sv, u);
                if constexpr (MODE == kFarPhi) {
                    o[0][k] = add_inv_root(xm, add_inv_root(xp, o[0][k]));
                } else {
                    const T r3p = inv_cube(xp), r3m = inv_cube(xm);
                    const T sum = r3p + r3m, dif = r3p - r3m;
                    sg[k] = fma(w, sum, sg[k]);
                    sa[k] = pi == 1 ? sv * dif : fma(sv, dif, sa[k]);
                    o[0][k] = fma(s2, sum, o[0][k]);
                }
            } else {
                const T u = C[k] + s2;
                const T xp = fma(mq[k], sv, u), xm = fma(-mq[k], sv, u);
                const T rp = rsqrt32(xp), rm = rsqrt32(xm);
                o[0][k] = fma(w, rp + rm, o[0][k]);
                if constexpr (MODE == kFarField) {
                    const T r3p = (rp * rp) * rp, r3m = (rm * rm) * rm;
                    sg[k] = fma(w, r3p + r3m, sg[k]);
                    SA[k] = fma(ws, r3p - r3m, SA[k]);
                }
            }
        }
    }
    if constexpr (MODE == kFarField) {
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            if constexpr (F64) {
                o[0][k] = fma(C[k], sg[k], fma(mq[k], sa[k], o[0][k]));
                SA[k] += sa[k];
            }
            o[1][k] = fma(da0[k], sg[k], o[1][k]);
            o[2][k] = fma(db[k], sg[k], o[2][k]);
            o[3][k] += sg[k];
        }
    }
}

// The 7 x 7 rule as seven pair rows; o (and SA) start at -0.0, the first row is peeled off.
template <int PPT, int MODE, typename T, typename T4>
__device__ __forceinline__ void pair_rows_sum(const T4* t, int base, const Local<PPT, T>& L,
                                              T (&o)[Sums<MODE>::kNode][PPT])
{
    T SA[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) SA[k] = T(-0.0);
    pair_row<PPT, MODE>(t, base, L, o, SA);
#pragma unroll 1
    for (int r = 1; r < 7; ++r) pair_row<PPT, MODE>(t, base + 4 * r, L, o, SA);
    if constexpr (MODE == kFarField) {
#pragma unroll
        for (int k = 0; k < PPT; ++k) o[1][k] -= SA[k];
    }
}

// One pair row for the gradient's sums (node_term, kFarGrad): with s5, s1, s2 the row's sums of
// w/r^5 times 1, the offset a - a0 and its square, the row adds s5, a0 s5 + s1, b s5,
// a0^2 s5 + 2 a0 s1 + s2, b (a0 s5 + s1) and the squares' sum.  12 instructions per node beside
// the reciprocal square root (16 with each node's own offset).  FP32 over D^2, as in node_term.
template <int PPT, typename T, typename T4>
__device__ __forceinline__ void grad_pair_row(const T4* t, int n0, const Local<PPT, T>& L, T (&o)[6][PPT])
{
    constexpr bool F64 = std::is_same<T, double>::value;
    const T4 hd = t[n0];
    const T b = hd.x, a0 = hd.y, wc = hd.z, g0 = hd.w;
    T C[PPT], mq[PPT], s5[PPT], s1[PPT], s2[PPT];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        C[k] = fma(L.q1[k], a0, fma(L.q2[k], b, grad_base(L, k, g0)));
        mq[k] = fma(T(2), F64 ? a0 : a0 * L.t[k], L.q1[k]);  // -2 (p1 - a0), over D^2 in FP32
        s5[k] = inv_fifth(wc, C[k]);
    }
#pragma unroll
    for (int pi = 1; pi <= 3; ++pi) {
        const T4 Q = t[n0 + pi];
        const T sv = Q.x, sq = Q.y, w = Q.z;
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            const T u = F64 ? C[k] + sq : fma(L.t[k], sq, C[k]);
            const T wp = inv_fifth(w, fma(mq[k], sv, u)), wm = inv_fifth(w, fma(-mq[k], sv, u));
            const T sum = wp + wm, dif = wp - wm;
            s5[k] += sum;
            s1[k] = pi == 1 ? sv * dif : fma(sv, dif, s1[k]);
            s2[k] = pi == 1 ? sq * sum : fma(sq, sum, s2[k]);
        }
    }
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const T ra = fma(a0, s5[k], s1[k]), rb = b * s5[k], raa = fma(a0, ra + s1[k], s2[k]);
        o[0][k] += s5[k];
        o[1][k] += ra;
        o[2][k] += rb;
        o[3][k] += raa;
        o[4][k] = fma(b, ra, o[4][k]);
        o[5][k] = fma(b, rb, o[5][k] + raa);
    }
}

// A compiled triangle rule with its orbit structure for the gradient's sums: on the S21 orbits
// per vertex T = sum w s/r^5 and Q = sum w s^2/r^5 (12 instructions per node beside the reciprocal
// square root), turned into the in-plane sums with the vertex u_k before the other orbits add.
template <int NN, int PPT, typename Lds, typename T>
__device__ __forceinline__ void tri_grad_sum(const Lds& s, int j, int base, const Local<PPT, T>& L, T (&o)[6][PPT])
{
    using O = TriOrbits<NN>;
    constexpr int NC = O::nc, N21 = O::n21, GS = O::gs, NG = NN - NC - 3 * N21;
    if constexpr (NC > 0) {
        const T w = s.nd[base].w;
#pragma unroll
        for (int k = 0; k < PPT; ++k) o[0][k] += inv_fifth(w, grad_base(L, k, T(0)));
    }
    if constexpr (N21 > 0) {
        const T u[3][2] = { { s.lc[0][j], s.lc[1][j] }, { s.lc[2][j], s.lc[3][j] }, { s.lc[4][j], s.lc[5][j] } };
        T Pk[3][PPT], Tk[3][PPT], Qk[3][PPT];
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            Pk[0][k] = fma(u[0][0], L.q1[k], u[0][1] * L.q2[k]);
            Pk[1][k] = fma(u[1][0], L.q1[k], u[1][1] * L.q2[k]);
            Pk[2][k] = -(Pk[0][k] + Pk[1][k]);
#pragma unroll
            for (int c = 0; c < 3; ++c) Tk[c][k] = Qk[c][k] = T(-0.0);
        }
#pragma unroll 1
        for (int ob = 0; ob < N21; ++ob) {
#pragma unroll
            for (int kk = 0; kk < 3; ++kk) {
                const auto Q = s.nd[base + NC + 3 * ob + kk];  // (s, |n|^2, s^2, w)
#pragma unroll
                for (int k = 0; k < PPT; ++k) {
                    const T w5 = inv_fifth(Q.w, fma(Q.x, Pk[kk][k], grad_base(L, k, Q.y)));
                    o[0][k] += w5;
                    Tk[kk][k] = fma(w5, Q.x, Tk[kk][k]);
                    Qk[kk][k] = fma(w5, Q.z, Qk[kk][k]);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < PPT; ++k)
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const T ta = u[c][0] * Qk[c][k], tb = u[c][1] * Qk[c][k];
                o[1][k] = fma(u[c][0], Tk[c][k], o[1][k]);
                o[2][k] = fma(u[c][1], Tk[c][k], o[2][k]);
                o[3][k] = fma(u[c][0], ta, o[3][k]);
                o[4][k] = fma(u[c][1], ta, o[4][k]);
                o[5][k] = fma(u[c][0], ta, fma(u[c][1], tb, o[5][k]));
            }
    }
    if constexpr (NG > 0) {
        const int g0 = base + NC + 3 * N21;
#pragma unroll 1
        for (int g = 0; g < NG / GS; ++g) {
#pragma unroll
            for (int u = 0; u < GS; ++u) node_term<PPT, kFarGrad, false>(s.nd[g0 + g * GS + u], L, o);
        }
    }
}

// One folded node whose r^2 / w^2 is x: potential (and field sums S3 and, for S21 nodes, the
// vertex sum tv = sum (w/r)^3 s / w^2, from which S1 and S2 follow per pair).
template <int MODE, typename T>
__device__ __forceinline__ void folded_point(T x, T iw2, T sv, T& o0, T& o3, T& tv)
{
    if constexpr (MODE == kFarPhi) {
        if constexpr (std::is_same<T, double>::value) o0 = add_inv_root(x, o0);
        else o0 += rsqrt32(x);
    } else {
        const T wr3 = inv_cube_phi(x, o0);
        tv = fma(wr3, sv, tv);
        o3 = fma(wr3, iw2, o3);
    }
}

// A compiled triangle rule with its orbit structure (TriOrbits), folded nodes: the centroid
// (r^2 = D^2), the S21 orbits (r^2 = D^2 + |n|^2 + s P_k with P_k = -2 d.u_k per pair; the
// field's in-plane sums per vertex), then the other orbits with the expanded form of
// node_term.  The sums in o start at -0.0; the first orbit of each kind is peeled off.
template <int NN, int PPT, int MODE, typename Lds, typename T>
__device__ __forceinline__ void tri_sum(const Lds& s, int j, int base, const Local<PPT, T>& L,
                                        T (&o)[Sums<MODE>::kNode][PPT])
{
    using O = TriOrbits<NN>;
    constexpr int NC = O::nc, N21 = O::n21, GS = O::gs, NG = NN - NC - 3 * N21;
    static_assert(NG % GS == 0, "orbit groups");
    constexpr int I3 = MODE == kFarPhi ? 0 : 3;  // index of S3 (unused for the potential alone)
    T Pk[3][PPT], Tk[3][PPT], dummy[PPT];
    if constexpr (N21 > 0) {
        const T ax = s.lc[0][j], ay = s.lc[1][j], bx = s.lc[2][j], by = s.lc[3][j];
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            Pk[0][k] = fma(ax, L.q1[k], ay * L.q2[k]);
            Pk[1][k] = fma(bx, L.q1[k], by * L.q2[k]);
            Pk[2][k] = -(Pk[0][k] + Pk[1][k]);
#pragma unroll
            for (int c = 0; c < 3; ++c) Tk[c][k] = T(-0.0);
        }
    }
    if constexpr (NC > 0) {
        const T iw2 = s.nd[base].z;
#pragma unroll
        for (int k = 0; k < PPT; ++k)
            folded_point<MODE, T>(L.H[k] * iw2, iw2, T(0), o[0][k], o[I3][k], dummy[k]);
    }
    if constexpr (N21 > 0) {
        auto orbit = [&](int ob) {
#pragma unroll
            for (int kk = 0; kk < 3; ++kk) {
                const auto Q = s.nd[base + NC + 3 * ob + kk];
#pragma unroll
                for (int k = 0; k < PPT; ++k)
                    folded_point<MODE, T>(fma(Q.x, Pk[kk][k], fma(L.H[k], Q.z, Q.y)), Q.z, Q.x, o[0][k], o[I3][k],
                                       Tk[kk][k]);
            }
        };
        orbit(0);
#pragma unroll 1
        for (int ob = 1; ob < N21; ++ob) orbit(ob);
    }
    if constexpr (NG > 0) {
        const int g0 = base + NC + 3 * N21;
        auto group = [&](int g) {
#pragma unroll
            for (int u = 0; u < GS; ++u) node_term<PPT, MODE, true>(s.nd[g0 + g * GS + u], L, o);
        };
        group(0);
#pragma unroll 1
        for (int g = 1; g < NG / GS; ++g) group(g);
    }
    if constexpr (N21 > 0 && MODE == kFarField) {
        const T l0 = s.lc[0][j], l1 = s.lc[1][j], l2 = s.lc[2][j], l3 = s.lc[3][j], l4 = s.lc[4][j], l5 = s.lc[5][j];
#pragma unroll
        for (int k = 0; k < PPT; ++k) {
            o[1][k] = fma(l0, Tk[0][k], fma(l2, Tk[1][k], fma(l4, Tk[2][k], o[1][k])));
            o[2][k] = fma(l1, Tk[0][k], fma(l3, Tk[1][k], fma(l5, Tk[2][k], o[2][k])));
        }
    }
}

// Sums of one element over its nodes [base, base + n) of the tile (Eq. 4.1, unit element
// charge) in the precision T of the tile (FP64, or FP32 for the mixed path).  NN > 0:
// compile-time node count; G > 0: tensor rule in groups of G (rows form).  Field, expanded:
// (sum w/r, S1, S2, S3) in node coordinates; rows: (sum w/r, local E1, local E2 without p3,
// sum w/r^3).  Gradient: the six sums of node_term.
template <int NN, int G, bool FOLD, bool TRI, int PPT, int MODE, typename Lds, typename T>
__device__ __forceinline__ void element_sum(const Lds& s, int j, int base, int n, const Local<PPT, T>& L,
                                            T (&o)[Sums<MODE>::kNode][PPT])
{
    constexpr int S = Sums<MODE>::kNode;
#pragma unroll
    for (int c = 0; c < S; ++c)
#pragma unroll
        for (int k = 0; k < PPT; ++k) o[c][k] = T(-0.0);
    const int nn = NN > 0 ? NN : n;
    if constexpr (G > 0) {
        static_assert(G == 7, "pair rows are built for the 7 x 7 rule");
        if constexpr (MODE == kFarGrad) {
#pragma unroll 1
            for (int r = 0; r < 7; ++r) grad_pair_row<PPT>(s.nd, base + 4 * r, L, o);
        } else {
            pair_rows_sum<PPT, MODE>(s.nd, base, L, o);
        }
    } else if constexpr (TRI && NN > 0 && MODE == kFarGrad) {
        tri_grad_sum<NN, PPT>(s, j, base, L, o);
    } else if constexpr (TRI && FOLD && NN > 0) {
        tri_sum<NN, PPT, MODE>(s, j, base, L, o);
    } else {
        node_term<PPT, MODE, FOLD>(s.nd[base], L, o);
        for_nodes<NN>(nn, [&](int i) { node_term<PPT, MODE, FOLD>(s.nd[base + i], L, o); });
    }
}

// Offsets of the lane's points from element j of the tile: D^2 in FP64 (the distance test,
// Sec. 2) and the coordinates the node sums need, in their precision.  Expanded: -2 f1.d,
// -2 f2.d and |p|^2 = D^2 (the rotation keeps the length, to rounding); rows: p = F d, and the
// expanded coordinates from them.  GRAD: in FP32 also 1/D and 1/D^2, and -2p over D^2 (grad_base).
template <int FR, bool GRAD, int PPT, typename Lds, typename T>
__device__ __forceinline__ void to_frame(const Lds& s, int j, const double (&x)[PPT], const double (&y)[PPT],
                                         const double (&z)[PPT], double (&D2)[PPT], Local<PPT, T>& L)
{
    const double cx = s.cx[j], cy = s.cy[j], cz = s.cz[j];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const double dx = x[k] - cx, dy = y[k] - cy, dz = z[k] - cz;
        L.dx[k] = dx;
        L.dy[k] = dy;
        L.dz[k] = dz;
        D2[k] = fma(dx, dx, fma(dy, dy, dz * dz));
        const T u = (T)dx, v = (T)dy, w = (T)dz;
        L.H[k] = (T)D2[k];
        if constexpr (FR == kFrExp) {
            L.q1[k] = fma(u, s.fr[0][j], fma(v, s.fr[1][j], w * s.fr[2][j]));
            L.q2[k] = fma(u, s.fr[3][j], fma(v, s.fr[4][j], w * s.fr[5][j]));
            if constexpr (GRAD) {
                T f = T(-2);
                if constexpr (std::is_same<T, float>::value) {
                    L.ri0[k] = rsqrt32(L.H[k]);
                    L.t[k] = L.ri0[k] * L.ri0[k];
                    f *= L.t[k];
                }
                L.q1[k] *= f;
                L.q2[k] *= f;
            }
        } else {
            L.p1[k] = fma(u, s.fr[0][j], fma(v, s.fr[1][j], w * s.fr[2][j]));
            L.p2[k] = fma(u, s.fr[3][j], fma(v, s.fr[4][j], w * s.fr[5][j]));
            L.p3[k] = fma(u, s.fr[6][j], fma(v, s.fr[7][j], w * s.fr[8][j]));
            L.q1[k] = T(-2) * L.p1[k];
            L.q2[k] = T(-2) * L.p2[k];
        }
    }
}

// The gradient's tensor in global axes from an element's sums (S5 ... Sg of node_term) and sum w/r^3
// (s3): out += q (delta_ij s3 - 3 M_ij), see add_element.
template <typename T>
__device__ __forceinline__ void add_grad(const T (&f1)[3], const T (&f2)[3], const T (&d)[3], T s3, T S5, T Sa, T Sb,
                                         T Saa, T Sab, T Sg, double q, double (&out)[6])
{
    const T Sbb = Sg - Saa;
    T v[3], z[3], g1[3], g2[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        v[c] = fma(f1[c], Sa, f2[c] * Sb);
        z[c] = fma(S5, d[c], -v[c]);
        g1[c] = fma(f1[c], Saa, f2[c] * Sab);
        g2[c] = fma(f1[c], Sab, f2[c] * Sbb);
    }
    auto M = [&](int u, int w) -> double {
        return (double)fma(d[u], z[w], fma(-v[u], d[w], fma(f1[u], g1[w], f2[u] * g2[w])));
    };
#pragma unroll
    for (int c = 0; c < 3; ++c) out[c] = fma(q, fma(-3.0, M(c, c), (double)s3), out[c]);
    out[3] = fma(-3.0 * q, M(0, 1), out[3]);
    out[4] = fma(-3.0 * q, M(0, 2), out[4]);
    out[5] = fma(-3.0 * q, M(1, 2), out[5]);
}

// acc += the element's contribution to point k (charge q, sums o), in FP64.
//   potential alone: phi += q sum w/r;
//   expanded sums:  phi += q sum w/r;  E += (q S3) d - (q f1) S1 - (q f2) S2;
//   rows:           phi += q sum w/r;  E += (q f1) E1 + (q f2) E2 + (q f3) p3 S3;
//   gradient:       dE_i/dx_j += q (delta_ij sum w/r^3 - 3 M_ij) with M = sum w (d - n)(d - n)^T / r^5
//                   over the nodes n = a f1 + b f2: M_ij = d_i z_j - v_i d_j + N_ij, v = Sa f1 + Sb f2,
//                   z = S5 d - v, N the in-plane second moments; sum w/r^3 from r^2 = D^2 + q1 a + q2 b +
//                   a^2 + b^2.  About 45 instructions per pair; rotating a local tensor takes twice
//                   that.  FP32: over D (d, v) and D^2 (N), the charge carrying 1/D^3.
template <int FR, int PPT, int MODE, typename Lds, typename T>
__device__ __forceinline__ void add_element(PointSet<PPT, MODE>& P, int k, double q, const Lds& s, int j,
                                            const Local<PPT, T>& L, const T (&o)[Sums<MODE>::kNode][PPT])
{
    if constexpr (MODE == kFarPhi) {
        P.acc[0][k] = fma(q, (double)o[0][k], P.acc[0][k]);
    } else if constexpr (MODE == kFarField) {
        P.acc[0][k] = fma(q, (double)o[0][k], P.acc[0][k]);
        if constexpr (FR == kFrExp) {
            const double s1 = (double)o[1][k], s2 = (double)o[2][k], qs3 = q * (double)o[3][k];
            P.acc[1][k] = fma(qs3, L.dx[k], fma(s.qr[0][j], s1, fma(s.qr[3][j], s2, P.acc[1][k])));
            P.acc[2][k] = fma(qs3, L.dy[k], fma(s.qr[1][j], s1, fma(s.qr[4][j], s2, P.acc[2][k])));
            P.acc[3][k] = fma(qs3, L.dz[k], fma(s.qr[2][j], s1, fma(s.qr[5][j], s2, P.acc[3][k])));
        } else {
            const double e1 = (double)o[1][k], e2 = (double)o[2][k], e3 = (double)(L.p3[k] * o[3][k]);
#pragma unroll
            for (int c = 0; c < 3; ++c)
                P.acc[1 + c][k] = fma(s.qr[c][j], e1, fma(s.qr[3 + c][j], e2, fma(s.qr[6 + c][j], e3, P.acc[1 + c][k])));
        }
    } else {
        T S5 = o[0][k], Sa = o[1][k], Sb = o[2][k], Saa = o[3][k], Sab = o[4][k], Sg = o[5][k];
        T d[3] = { (T)L.dx[k], (T)L.dy[k], (T)L.dz[k] };
        T s3;
        if constexpr (std::is_same<T, double>::value) {
            s3 = fma(L.H[k], S5, fma(L.q1[k], Sa, fma(L.q2[k], Sb, Sg)));
        } else {
            const T ri0 = L.ri0[k], t = L.t[k];
            Sg *= t;
            s3 = S5 + fma(L.q1[k], Sa, fma(L.q2[k], Sb, Sg));
            Sa *= ri0; Sb *= ri0; Saa *= t; Sab *= t;
            d[0] *= ri0; d[1] *= ri0; d[2] *= ri0;
            q *= (double)ri0 * (double)t;  // (1/D^3 would leave FP32's range below 1e-13 of a unit)
        }
        const T f1[3] = { s.fr[0][j], s.fr[1][j], s.fr[2][j] }, f2[3] = { s.fr[3][j], s.fr[4][j], s.fr[5][j] };
        double out[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) out[c] = P.acc[c][k];
        add_grad(f1, f2, d, s3, S5, Sa, Sb, Saa, Sab, Sg, q, out);
#pragma unroll
        for (int c = 0; c < 6; ++c) P.acc[c][k] = out[c];
    }
}

// group size of the rows form for a rectangle rule of NN nodes (7 x 7 only)
template <bool TRI, int NN>
constexpr int tensor_group() { return (!TRI && NN == 49) ? 7 : 0; }

// frame form of an element kind with a compiled rule of NN nodes
template <bool TRI, int NN, int MODE>
constexpr int frame_form() { return (MODE == kFarField && tensor_group<TRI, NN>() > 0) ? kFrRows : kFrExp; }

// One element kind over [e_begin, e_end) with one rule; NN > 0 is the compile-time node
// count, NN == 0 reads it at run time.  FOLD: the rule's weights are all positive (the
// nodes are staged divided by w^2).
template <int NN, bool TRI, bool MIXED, int PPT, int MODE, bool FOLD, typename Lds>
__device__ __forceinline__ void far_eval_range(const FarArgs& a, Lds& s, PointSet<PPT, MODE>& P, int64_t e_begin,
                                               int64_t e_end)
{
    using T = typename Lds::T;
    constexpr int FR = frame_form<TRI, NN, MODE>();
    constexpr bool GRAD = MODE == kFarGrad;
    constexpr bool FOLD_ = FOLD && !GRAD && tensor_group<TRI, NN>() == 0;
    constexpr bool ORBITS = FOLD_ || (GRAD && TRI && NN > 0);
    const int nn = NN > 0 ? NN : (TRI ? a.rules.nt : a.rules.nr);
    const int TE = tile_elems<Lds>(nn);
    const TriForms tf = fixed_forms<NN, TRI && ORBITS>(nn);
    for (int64_t t0 = e_begin; t0 < e_end; t0 += TE) {
        const int te = (int)min((int64_t)TE, e_end - t0);
        __syncthreads();
        stage_tile<TRI, MIXED, FR, MODE == kFarField, GRAD>(s, a.el, a.rules, nn, t0, te, a.rhs, 1,
                                                               ORBITS ? nn : 0, tensor_group<TRI, NN>() > 0 ? 0 : nn,
                                                               tf, sum_scale<MODE, T>());
        __syncthreads();
        for (int j = 0; j < te; ++j) {
            const double thr2 = s.thr2[j], q = s.q[0][j];
            double D2[PPT];
            Local<PPT, T> L;
            to_frame<FR, GRAD>(s, j, P.x, P.y, P.z, D2, L);
            bool nr[PPT];
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                nr[k] = P.valid[k] && (D2[k] < thr2);  // listed by near_list_kernel
            }
            T o[Sums<MODE>::kNode][PPT];
            element_sum<NN, tensor_group<TRI, NN>(), FOLD_, TRI, PPT, MODE>(s, j, j * nn, nn, L, o);
#pragma unroll
            for (int k = 0; k < PPT; ++k)
                if (!nr[k]) add_element<FR, PPT, MODE>(P, k, q, s, j, L, o);
        }
    }
}

// Expanded sums (node coordinates) of a rectangle level turned into the local field of the
// rows form: E1 = p1 S3 - S1, E2 = p2 S3 - S2.
template <int PPT, typename T>
__device__ __forceinline__ void exp_to_rows(const Local<PPT, T>& L, T (&o)[4][PPT])
{
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        o[1][k] = fma(L.p1[k], o[3][k], -o[1][k]);
        o[2][k] = fma(L.p2[k], o[3][k], -o[2][k]);
    }
}

// One element kind with the rule chosen by distance ratio (Sec. 4): the staged nodes of an
// element are the four levels back to back; a pair needs level l when D^2 >= c[l] (near_dr
// L)^2 (the last level otherwise).  The wavefront runs the finest level that any of its
// pairs needs, once, for all its lanes: a finer rule is at least as accurate at a larger
// distance ratio, and one level per wavefront costs less than each level a lane needs.
// N0..N3 > 0: compile-time counts (the levels' weights are then all positive).
// Triangles take the expanded form throughout; rectangles the rows form for a 7 x 7 last
// level, the expanded form (turned into the rows form's local field) for the others.
// Terms summed by the wavefront (w: pairs at each wavefront level) and at the pairs' own
// levels (n: pairs at levels 0, 1, 2 of nc in all), the levels having o1, o2 - o1, o3 - o2 and
// nn - o3 nodes.
__device__ __forceinline__ void add_terms(unsigned w0, unsigned w1, unsigned w2, unsigned w3, unsigned nc,
                                          unsigned n0, unsigned n1, unsigned n2, int o1, int o2, int o3, int nn,
                                          unsigned long long& terms, unsigned long long& terms_pair)
{
    terms += (unsigned long long)w0 * (unsigned)o1 + (unsigned long long)w1 * (unsigned)(o2 - o1) +
             (unsigned long long)w2 * (unsigned)(o3 - o2) + (unsigned long long)w3 * (unsigned)(nn - o3);
    terms_pair += (unsigned long long)n0 * (unsigned)o1 + (unsigned long long)n1 * (unsigned)(o2 - o1) +
                  (unsigned long long)n2 * (unsigned)(o3 - o2) +
                  (unsigned long long)(nc - n0 - n1 - n2) * (unsigned)(nn - o3);
}

template <int N0, int N1, int N2, int N3, bool TRI, bool MIXED, int PPT, int MODE, typename Lds>
__device__ __forceinline__ void far_eval_dr_range(const FarArgs& a, Lds& s, PointSet<PPT, MODE>& P, int64_t e_begin,
                                                  int64_t e_end, unsigned long long& terms,
                                                  unsigned long long& terms_pair)
{
    using T = typename Lds::T;
    constexpr bool GRAD = MODE == kFarGrad;
    constexpr int FR = (TRI || MODE != kFarField) ? kFrExp : kFrRows;
    constexpr bool FOLD = N0 > 0 && !GRAD;
    const int* off = TRI ? a.lv.tri_off : a.lv.rect_off;
    const double* c = TRI ? a.lv.tri_c : a.lv.rect_c;
    constexpr bool FIXED = N0 > 0;  // the levels' sizes are known
    const int o1 = FIXED ? N0 : off[1], o2 = FIXED ? N0 + N1 : off[2], o3 = FIXED ? N0 + N1 + N2 : off[3];
    const int nn = FIXED ? N0 + N1 + N2 + N3 : off[4];
    const double c0 = c[0], c1 = c[1], c2 = c[2];
    const double c_all = fmax(c0, 1.0);  // (a level's limit may lie below the near one's: no near pair passes)
    const int TE = tile_elems<Lds>(nn);
    TriForms tf{ 4, { 0, o1, o2, o3, nn }, { 0, 0, 0, 0 }, { 0, 0, 0, 0 } };
    if (TRI && N0 > 0) {
        tf.nc[0] = TriOrbits<N0>::nc; tf.n21[0] = 3 * TriOrbits<N0>::n21;
        tf.nc[1] = TriOrbits<N1>::nc; tf.n21[1] = 3 * TriOrbits<N1>::n21;
        tf.nc[2] = TriOrbits<N2>::nc; tf.n21[2] = 3 * TriOrbits<N2>::n21;
        tf.nc[3] = TriOrbits<N3>::nc; tf.n21[3] = 3 * TriOrbits<N3>::n21;
    }
    unsigned long long vmask[PPT];  // the lanes with a point, per point of the lane
#pragma unroll
    for (int k = 0; k < PPT; ++k) vmask[k] = lane_mask(P.valid[k]);
    unsigned n_valid = 0;
#pragma unroll
    for (int k = 0; k < PPT; ++k) n_valid += (unsigned)__popcll(vmask[k]);
    for (int64_t t0 = e_begin; t0 < e_end; t0 += TE) {
        const int te = (int)min((int64_t)TE, e_end - t0);
        // the tile's pair counts (scalar, 32 bits: at most 64 PPT TE per tile): summed by the
        // wavefront at each of its levels, and at the pairs' own levels (all, level 0, 1, 2)
        unsigned w0 = 0, w1 = 0, w2 = 0, w3 = 0, nc = 0, n0 = 0, n1 = 0, n2 = 0;
        __syncthreads();
        // the 7 x 7 last level of the rectangles keeps its weights (rows form)
        const int nfold = N0 == 0 ? 0 : (tensor_group<TRI, N3>() > 0 ? o3 : nn);
        const int prow = tensor_group<TRI, N3>() > 0 ? o3 : nn;
        stage_tile<TRI, MIXED, FR, MODE == kFarField, GRAD>(s, a.el, a.lv.tab, nn, t0, te, a.rhs, 1, nfold, prow, tf,
                                             sum_scale<MODE, T>());
        __syncthreads();
        // (a wavefront without a point only helps staging: a served batch of 64 points or fewer has three
        // such of four, and the first test below is true for them)
        if (n_valid == 0) continue;
        for (int j = 0; j < te; ++j) {
            const double thr2 = s.thr2[j], q = s.q[0][j];
            double D2[PPT];
            Local<PPT, T> L;
            to_frame<FR, GRAD>(s, j, P.x, P.y, P.z, D2, L);
            // the level each pair's distance ratio asks for, as wavefront masks straight from the
            // comparisons: pairs for which level 0 suffices, then level 1, level 2, and every far
            // pair (near pairs are listed by near_list_kernel and contribute nothing here); the
            // wavefront's level and the term counts are then scalar work on the masks
            {
                // the common case first: level 0 for every pair and none near: one comparison a pair
                // instead of four, and nothing masked
                const double all0 = c_all * thr2;
                unsigned long long short_of = 0;
#pragma unroll
                for (int k = 0; k < PPT; ++k) short_of |= vmask[k] & ~lane_mask(D2[k] >= all0);
                if (short_of == 0) {
                    T o[Sums<MODE>::kNode][PPT];
                    element_sum<N0, 0, FOLD, TRI, PPT, MODE>(s, j, j * nn, o1, L, o);
                    if constexpr (FR == kFrRows) exp_to_rows<PPT>(L, o);
#pragma unroll
                    for (int k = 0; k < PPT; ++k) add_element<FR, PPT, MODE>(P, k, q, s, j, L, o);
                    nc += n_valid; n0 += n_valid; w0 += n_valid;
                    continue;
                }
            }
            const double lim0 = c0 * thr2, lim1 = c1 * thr2, lim2 = c2 * thr2;
            bool far[PPT];
            unsigned long long u0 = 0, u1 = 0, u2 = 0, u3 = 0;  // the lanes with a pair at each level
            unsigned ec = 0;                                      // the element's far pairs
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                // masks of plain comparisons only (the backend turns a mask of a combined
                // condition into a vector select and another comparison); the rest is scalar
                far[k] = P.valid[k] && !(D2[k] < thr2);
                const unsigned long long mf = vmask[k] & ~lane_mask(D2[k] < thr2);
                const unsigned long long m0 = mf & lane_mask(D2[k] >= lim0);
                const unsigned long long m1 = mf & lane_mask(D2[k] >= lim1) & ~m0;
                const unsigned long long m2 = mf & lane_mask(D2[k] >= lim2) & ~(m0 | m1);
                u0 |= m0; u1 |= m1; u2 |= m2; u3 |= mf & ~(m0 | m1 | m2);
                ec += (unsigned)__popcll(mf);
                n0 += (unsigned)__popcll(m0);
                n1 += (unsigned)__popcll(m1);
                n2 += (unsigned)__popcll(m2);
            }
            // the finest level any pair of the wavefront needs
            const int wl = u3 ? 3 : (u2 ? 2 : (u1 ? 1 : (u0 ? 0 : -1)));
            if (wl < 0) continue;
            nc += ec;
            T o[Sums<MODE>::kNode][PPT];
            const int b = j * nn;
            if (wl == 0) { element_sum<N0, 0, FOLD, TRI, PPT, MODE>(s, j, b, o1, L, o); w0 += ec; }
            else if (wl == 1) { element_sum<N1, 0, FOLD, TRI, PPT, MODE>(s, j, b + o1, o2 - o1, L, o); w1 += ec; }
            else if (wl == 2) { element_sum<N2, 0, FOLD, TRI, PPT, MODE>(s, j, b + o2, o3 - o2, L, o); w2 += ec; }
            else {
                constexpr int G3 = tensor_group<TRI, N3>();
                element_sum<N3, G3, FOLD && (TRI || G3 == 0), TRI, PPT, MODE>(s, j, b + o3, nn - o3, L, o);
                w3 += ec;
            }
            if constexpr (FR == kFrRows) {
                // rows form for the rotation back; the 7 x 7 last level is in it already
                if (!(wl == 3 && tensor_group<TRI, N3>() > 0)) exp_to_rows<PPT>(L, o);
            }
#pragma unroll
            for (int k = 0; k < PPT; ++k)
                if (far[k]) add_element<FR, PPT, MODE>(P, k, q, s, j, L, o);
        }
        add_terms(w0, w1, w2, w3, nc, n0, n1, n2, o1, o2, o3, nn, terms, terms_pair);
    }
}

// The wavefronts' term counts (the same in every lane) added up over the workgroup: one atomic per
// counter and workgroup.
__device__ __forceinline__ void add_block_terms(unsigned long long terms, unsigned long long terms_pair, DevCounters* ctr)
{
    __shared__ unsigned long long sums[2];
    if (threadIdx.x < 2) sums[threadIdx.x] = 0ull;
    __syncthreads();
    if (lane_id() == 0) {
        atomicAdd(&sums[0], terms);
        atomicAdd(&sums[1], terms_pair);
    }
    __syncthreads();
    if (threadIdx.x == 0 && sums[0]) {
        atomicAdd(&ctr->node_ints, sums[0]);
        atomicAdd(&ctr->node_ints_pair, sums[1]);
    }
}

// DR == false: one rule per kind, NT / NR nodes.  DR == true: levels (T0..T3 / R0..R3).
// MODE: potential and field, potential alone, or the field gradient.  Compiled node counts (NT, NR > 0)
// are used only for rules whose weights are all positive (their nodes are folded).
template <bool DR, int NT, int NR, int T1, int T2, int T3, int R1, int R2, int R3, bool MIXED, int PPT, int MODE>
__global__ __launch_bounds__(kBlock) void far_eval_kernel(FarArgs a)
{
    constexpr int NO = Sums<MODE>::kOut;
    __shared__ TileLds<MIXED, 1, !MIXED && PPT == 1 && MODE != kFarGrad> s;
    PointSet<PPT, MODE> P;
    const int64_t base = (int64_t)blockIdx.x * (kBlock * PPT) + threadIdx.x;
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int64_t p = base + (int64_t)k * kBlock;
        P.valid[k] = p < a.n;
        P.idx[k] = (uint32_t)p;
        P.x[k] = P.valid[k] ? a.pts[p] : 0.0;
        P.y[k] = P.valid[k] ? a.pts[a.n + p] : 0.0;
        P.z[k] = P.valid[k] ? a.pts[2 * a.n + p] : 0.0;
#pragma unroll
        for (int c = 0; c < NO; ++c) P.acc[c][k] = 0.0;
    }
    int64_t e_lo = a.elem_begin, e_hi = a.elem_end;
    if (a.n_split > 1) {
        e_lo = min(a.elem_begin + (int64_t)blockIdx.y * a.chunk, a.elem_end);
        e_hi = min(e_lo + a.chunk, a.elem_end);
    }
    const int64_t nt_end = min((int64_t)a.el.n_tri, e_hi);
    const int64_t nr_begin = max((int64_t)a.el.n_tri, e_lo);
    if (DR) {
        unsigned long long terms = 0, terms_pair = 0;
        if (e_lo < nt_end)
            far_eval_dr_range<NT, T1, T2, T3, true, MIXED, PPT, MODE>(a, s, P, e_lo, nt_end, terms, terms_pair);
        if (nr_begin < e_hi)
            far_eval_dr_range<NR, R1, R2, R3, false, MIXED, PPT, MODE>(a, s, P, nr_begin, e_hi, terms, terms_pair);
        add_block_terms(terms, terms_pair, a.ctr);
    } else {
        if (e_lo < nt_end) far_eval_range<NT, true, MIXED, PPT, MODE, (NT > 0)>(a, s, P, e_lo, nt_end);
        if (nr_begin < e_hi) far_eval_range<NR, false, MIXED, PPT, MODE, (NR > 0)>(a, s, P, nr_begin, e_hi);
    }
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        if (!P.valid[k]) continue;
        const int64_t p = base + (int64_t)k * kBlock;
        if (a.partial) {  // element-split launch: unscaled partial sums, reduced later in fixed order
            double* o = a.partial + (int64_t)blockIdx.y * NO * a.n;
#pragma unroll
            for (int c = 0; c < NO; ++c) o[c * a.n + p] = P.acc[c][k];
        } else if (MODE == kFarGrad) {
#pragma unroll
            for (int c = 0; c < NO; ++c) a.G[c * a.n + p] = a.K * P.acc[c][k];
        } else {
            a.phi[p] = a.K * P.acc[0][k];
            if (MODE == kFarField && a.E) {
                a.E[p] = a.K * P.acc[NO > 1 ? 1 : 0][k];
                a.E[a.n + p] = a.K * P.acc[NO > 2 ? 2 : 0][k];
                a.E[2 * a.n + p] = a.K * P.acc[NO > 3 ? 3 : 0][k];
            }
        }
    }
}

// ------------------------------------------------------------ far field: few points -----
// A handful of points: an element per lane instead of a point per lane.  With one point the lanes
// of far_eval_kernel's wavefronts would be idle but one, and a workgroup's chunk of elements a
// serial chain (150,000 elements, rules by distance ratio: far kernel 5,700 us, 14 us so).  Each lane
// takes its element's record from memory, forms the Gaussian points of the rule (from LDS, the
// same node for the whole wavefront) in the element's frame and sums them for PF points, all in
// FP64 whatever the precision asked for: a launch of this size waits for latency, not for
// arithmetic.  The near pairs go to the list here, so that there is no list pass.  The lanes' sums
// are added by a fixed butterfly, the wavefronts' in order: chunk partial sums as those of a split
// launch.
template <bool DR, int PF, int MODE>
struct FewRange {
    static constexpr int NO = Sums<MODE>::kOut, NS = Sums<MODE>::kNode;
    double x[PF], y[PF], z[PF];
    bool valid[PF];
    uint32_t idx[PF];
    double acc[NO][PF];
    unsigned long long terms, terms_pair;

    template <bool TRI>
    __device__ __forceinline__ void run(const FarArgs& a, const double4* __restrict__ nodes, int64_t lo, int64_t hi)
    {
        const Elements& el = a.el;
        const int64_t ne = el.ne;
        const int* off = TRI ? a.lv.tri_off : a.lv.rect_off;
        const double* lim = TRI ? a.lv.tri_c : a.lv.rect_c;
        const int n_nodes = TRI ? a.rules.nt : a.rules.nr;
        for (int64_t e0 = lo; e0 < hi; e0 += kBlock) {  // (the same trips for every lane)
            const bool active = e0 + threadIdx.x < hi;
            const int64_t e = active ? e0 + threadIdx.x : hi - 1;
            const double c0 = el.cen[e], c1 = el.cen[ne + e], c2 = el.cen[2 * ne + e], thr2 = el.thr2[e];
            const double f1[3] = { el.frame[e], el.frame[ne + e], el.frame[2 * ne + e] };
            const double f2[3] = { el.frame[3 * ne + e], el.frame[4 * ne + e], el.frame[5 * ne + e] };
            double lc[6];
#pragma unroll
            for (int c = 0; c < (TRI ? 6 : 3); ++c) lc[c] = el.loc[(int64_t)c * ne + e];
            const double q = sum_scale<MODE, double>() * el.q[(int64_t)a.rhs * ne + e];
            double d[PF][3], H[PF], q1[PF], q2[PF], o[NS][PF];
            bool far[PF];
            int level = 0;  // of the lane's pairs
            bool any = false;
            unsigned long long pair_terms = 0;
            unsigned n_far = 0;
#pragma unroll
            for (int k = 0; k < PF; ++k) {
                d[k][0] = x[k] - c0; d[k][1] = y[k] - c1; d[k][2] = z[k] - c2;
                H[k] = fma(d[k][0], d[k][0], fma(d[k][1], d[k][1], d[k][2] * d[k][2]));
                q1[k] = -2.0 * fma(d[k][0], f1[0], fma(d[k][1], f1[1], d[k][2] * f1[2]));
                q2[k] = -2.0 * fma(d[k][0], f2[0], fma(d[k][1], f2[1], d[k][2] * f2[2]));
                const bool near = active && valid[k] && H[k] < thr2;
                append_near(near, idx[k], (uint32_t)e, a.near_list, a.near_cap, a.ctr);
                far[k] = active && valid[k] && !near;
                any |= far[k];
                if (DR && far[k]) {
                    const int l = H[k] >= lim[0] * thr2 ? 0 : (H[k] >= lim[1] * thr2 ? 1 : (H[k] >= lim[2] * thr2 ? 2 : 3));
                    level = max(level, l);
                    pair_terms += (unsigned)(off[l + 1] - off[l]);
                    ++n_far;
                }
#pragma unroll
                for (int c = 0; c < NS; ++c) o[c][k] = 0.0;
            }
            if (lane_mask(any) == 0ull) continue;
            int i_lo = 0, i_hi = n_nodes;
            if (DR) {  // the finest level any pair of the wavefront needs
                level = lane_mask(level >= 3) ? 3 : (lane_mask(level >= 2) ? 2 : (lane_mask(level >= 1) ? 1 : 0));
                i_lo = off[level];
                i_hi = off[level + 1];
                terms += (unsigned long long)n_far * (unsigned)(i_hi - i_lo);
                terms_pair += pair_terms;
            }
#pragma unroll 2
            for (int i = i_lo; i < i_hi; ++i) {
                const double4 R = nodes[i];
                double na, nb, w;
                if (TRI) {
                    na = fma(R.x, lc[0], fma(R.y, lc[2], R.z * lc[4]));
                    nb = fma(R.x, lc[1], fma(R.y, lc[3], R.z * lc[5]));
                    w = R.w;
                } else {
                    na = fma(R.x, lc[0], R.y * lc[2]);
                    nb = R.x * lc[1];
                    w = R.z;
                }
                const double g = fma(na, na, nb * nb);
#pragma unroll
                for (int k = 0; k < PF; ++k) {
                    const double r2 = fma(q1[k], na, fma(q2[k], nb, H[k] + g));
                    if constexpr (MODE == kFarPhi) {
                        o[0][k] = add_inv_root(w, r2, o[0][k]);
                    } else if constexpr (MODE == kFarField) {
                        const double w3 = inv_cube_phi(w, r2, o[0][k]);
                        o[1][k] = fma(w3, na, o[1][k]);
                        o[2][k] = fma(w3, nb, o[2][k]);
                        o[3][k] += w3;
                    } else {
                        const double w5 = inv_fifth(w, r2), ua = w5 * na;
                        o[0][k] += w5;
                        o[1][k] += ua;
                        o[2][k] = fma(w5, nb, o[2][k]);
                        o[3][k] = fma(ua, na, o[3][k]);
                        o[4][k] = fma(ua, nb, o[4][k]);
                        o[5][k] = fma(w5, g, o[5][k]);
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < PF; ++k) {
                if (!far[k]) continue;
                if constexpr (MODE == kFarGrad) {
                    const double s3 = fma(H[k], o[0][k], fma(q1[k], o[1][k], fma(q2[k], o[2][k], o[5][k])));
                    double out[6];
#pragma unroll
                    for (int c = 0; c < 6; ++c) out[c] = acc[c][k];
                    add_grad(f1, f2, d[k], s3, o[0][k], o[1][k], o[2][k], o[3][k], o[4][k], o[5][k], q, out);
#pragma unroll
                    for (int c = 0; c < 6; ++c) acc[c][k] = out[c];
                } else {
                    acc[0][k] = fma(q, o[0][k], acc[0][k]);
                    if constexpr (MODE == kFarField)
#pragma unroll
                        for (int c = 0; c < 3; ++c)
                            acc[1 + c][k] = fma(q, fma(o[3][k], d[k][c], -fma(f1[c], o[1][k], f2[c] * o[2][k])), acc[1 + c][k]);
                }
            }
        }
    }
};

template <bool DR, int PF, int MODE>
__global__ __launch_bounds__(kBlock) void far_few_kernel(FarArgs a)
{
    constexpr int NO = Sums<MODE>::kOut;
    extern __shared__ double4 few_nodes[];  // the rules' nodes (all levels): triangles, rectangles
    __shared__ double part[kBlock / 64][NO * PF];
    const RuleTables& R = DR ? a.lv.tab : a.rules;
    for (int i = threadIdx.x; i < R.nt + R.nr; i += kBlock) {
        const double* src = i < R.nt ? R.tri + 4 * i : R.rect + 4 * (i - R.nt);
        few_nodes[i] = make_double4(src[0], src[1], src[2], src[3]);
    }
    FewRange<DR, PF, MODE> F;
    F.terms = F.terms_pair = 0;
#pragma unroll
    for (int k = 0; k < PF; ++k) {
        const int64_t p = (int64_t)blockIdx.y * PF + k;
        F.valid[k] = p < a.n;
        F.idx[k] = (uint32_t)p;
        F.x[k] = F.valid[k] ? a.pts[p] : 0.0;
        F.y[k] = F.valid[k] ? a.pts[a.n + p] : 0.0;
        F.z[k] = F.valid[k] ? a.pts[2 * a.n + p] : 0.0;
#pragma unroll
        for (int c = 0; c < NO; ++c) F.acc[c][k] = 0.0;
    }
    __syncthreads();
    const int64_t lo = min((int64_t)blockIdx.x * a.chunk, a.el.ne), hi = min(lo + a.chunk, a.el.ne);
    const int64_t nt = a.el.n_tri;
    if (lo < nt) F.template run<true>(a, few_nodes, lo, min(hi, nt));
    if (hi > nt) F.template run<false>(a, few_nodes + R.nt, max(lo, nt), hi);
    // the lanes' sums by a fixed butterfly, the wavefronts' in order
    const int wave = threadIdx.x / 64;
#pragma unroll
    for (int c = 0; c < NO; ++c)
#pragma unroll
        for (int k = 0; k < PF; ++k) {
            double v = F.acc[c][k];
            for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
            if (lane_id() == 0) part[wave][c * PF + k] = v;
        }
    if (DR) {
        unsigned long long t = F.terms, tp = F.terms_pair;
        for (int o = 32; o > 0; o >>= 1) { t += __shfl_xor(t, o); tp += __shfl_xor(tp, o); }
        add_block_terms(t, tp, a.ctr);
    }
    __syncthreads();
    if (threadIdx.x < NO * PF) {
        const int c = threadIdx.x / PF, k = threadIdx.x % PF;
        const int64_t p = (int64_t)blockIdx.y * PF + k;
        double v = 0.0;
        for (int w = 0; w < kBlock / 64; ++w) v += part[w][threadIdx.x];
        if (p < a.n) a.partial[((int64_t)blockIdx.x * NO + c) * a.n + p] = v;
    }
}

// ------------------------------------------------------- far field: collocation -----
template <int NN, bool TRI, bool MIXED, int PPT, typename Lds>
__device__ __forceinline__ void far_colloc_range(const FarArgs& a, Lds& s, const double (&px)[PPT],
                                                 const double (&py)[PPT], const double (&pz)[PPT],
                                                 const bool (&valid)[PPT], const uint32_t (&idx)[PPT],
                                                 double (&acc)[PPT][kMaxRhs], int64_t e_begin, int64_t e_end)
{
    using T = typename Lds::T;
    constexpr int FR = frame_form<TRI, NN, kFarPhi>();
    constexpr bool FOLD = NN > 0 && tensor_group<TRI, NN>() == 0;
    const int nn = NN > 0 ? NN : (TRI ? a.rules.nt : a.rules.nr);
    const int TE = tile_elems<Lds>(nn);
    const int nrhs = a.n_rhs;
    const TriForms tf = fixed_forms<NN, TRI && FOLD>(nn);
    for (int64_t t0 = e_begin; t0 < e_end; t0 += TE) {
        const int te = (int)min((int64_t)TE, e_end - t0);
        __syncthreads();
        stage_tile<TRI, MIXED, FR, false, false>(s, a.el, a.rules, nn, t0, te, 0, nrhs, FOLD ? nn : 0,
                                                   tensor_group<TRI, NN>() > 0 ? 0 : nn, tf, sum_scale<kFarPhi, T>());
        __syncthreads();
        for (int j = 0; j < te; ++j) {
            const double thr2 = s.thr2[j];
            double D2[PPT];
            Local<PPT, T> L;
            to_frame<FR, false>(s, j, px, py, pz, D2, L);
            bool nr[PPT];
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                nr[k] = valid[k] && (D2[k] < thr2);  // listed by near_list_kernel
            }
            T o[1][PPT];
            element_sum<NN, tensor_group<TRI, NN>(), FOLD, TRI, PPT, kFarPhi>(s, j, j * nn, nn, L, o);
#pragma unroll
            for (int k = 0; k < PPT; ++k) {
                if (!nr[k]) {
                    const double v = (double)o[0][k];
#pragma unroll
                    for (int r = 0; r < kMaxRhs; ++r)
                        if (r < nrhs) acc[k][r] = fma(s.q[r][j], v, acc[k][r]);
                }
            }
        }
    }
}

template <int NT, int NR, bool MIXED, int PPT>
__global__ __launch_bounds__(kBlock) void far_colloc_kernel(FarArgs a)
{
    __shared__ TileLds<MIXED, kMaxRhs, false> s;
    const int64_t ne = a.el.ne;
    const int64_t base = (int64_t)blockIdx.x * (kBlock * PPT) + threadIdx.x;
    double px[PPT], py[PPT], pz[PPT];
    bool valid[PPT];
    uint32_t idx[PPT];
    double acc[PPT][kMaxRhs];
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        const int64_t p = base + (int64_t)k * kBlock;
        valid[k] = p < ne;
        idx[k] = (uint32_t)p;
        px[k] = valid[k] ? a.el.cen[p] : 0.0;
        py[k] = valid[k] ? a.el.cen[ne + p] : 0.0;
        pz[k] = valid[k] ? a.el.cen[2 * ne + p] : 0.0;
#pragma unroll
        for (int r = 0; r < kMaxRhs; ++r) acc[k][r] = 0.0;
    }
    int64_t e_lo = 0, e_hi = ne;
    if (a.n_split > 1) {
        e_lo = min((int64_t)blockIdx.y * a.chunk, ne);
        e_hi = min(e_lo + a.chunk, ne);
    }
    const int64_t nt = a.el.n_tri;
    const int64_t t_hi = min(nt, e_hi);
    if (e_lo < t_hi) far_colloc_range<NT, true, MIXED, PPT>(a, s, px, py, pz, valid, idx, acc, e_lo, t_hi);
    const int64_t r_lo = max(nt, e_lo);
    if (r_lo < e_hi) far_colloc_range<NR, false, MIXED, PPT>(a, s, px, py, pz, valid, idx, acc, r_lo, e_hi);
#pragma unroll
    for (int k = 0; k < PPT; ++k) {
        if (!valid[k]) continue;
        const int64_t p = base + (int64_t)k * kBlock;
        if (a.partial) {  // element chunk blockIdx.y: unscaled partial sums [split][rhs][ne]
            double* o = a.partial + (int64_t)blockIdx.y * a.n_rhs * ne;
#pragma unroll
            for (int r = 0; r < kMaxRhs; ++r)
                if (r < a.n_rhs) o[(int64_t)r * ne + p] = acc[k][r];
        } else {
#pragma unroll
            for (int r = 0; r < kMaxRhs; ++r)
                if (r < a.n_rhs) a.phi[(int64_t)r * ne + p] = a.K * acc[k][r];
        }
    }
}

// --------------------------------------------------------------- near field ---------
struct NearState {
    int kind;        // 0 triangle, 1 rectangle
    int level;       // 0 = the element itself
    int i, j;        // lattice position at this level
    bool up;         // triangle orientation (up: vertices (i,j),(i+1,j),(i,j+1))
};

// Index of a child within its parent and the parent's lattice position.
__device__ __forceinline__ int child_index(NearState& s)
{
    const int a = s.i & 1, b = s.j & 1;
    int c;
    bool pup = true;
    if (s.kind == 1) {
        c = a + 2 * b;
    } else if (s.up) {
        if (a && b) { pup = false; c = 3; }
        else c = a ? 1 : (b ? 2 : 0);
    } else {
        if (!a && !b) { pup = true; c = 3; }
        else { pup = false; c = (a && b) ? 0 : (b ? 1 : 2); }
    }
    s.i >>= 1;
    s.j >>= 1;
    s.up = pup;
    s.level -= 1;
    return c;
}

// Child c of the node s (s becomes the child).
__device__ __forceinline__ void to_child(NearState& s, int c)
{
    const int i2 = 2 * s.i, j2 = 2 * s.j;
    s.level += 1;
    if (s.kind == 1) {
        s.i = i2 + (c & 1);
        s.j = j2 + (c >> 1);
    } else if (s.up) {  // up parent: up(2i,2j), up(2i+1,2j), up(2i,2j+1), down(2i,2j)
        s.i = i2 + (c == 1 ? 1 : 0);
        s.j = j2 + (c == 2 ? 1 : 0);
        s.up = (c != 3);
    } else {  // down parent: down(2i+1,2j+1), down(2i,2j+1), down(2i+1,2j), up(2i+1,2j+1)
        s.i = i2 + (c == 1 ? 0 : 1);
        s.j = j2 + (c == 2 ? 0 : 1);
        s.up = (c == 3);
    }
}

// Move to the next node of the depth-first walk after finishing node s; false when the
// walk has returned to the root.
__device__ __forceinline__ bool advance(NearState& s)
{
    while (s.level > 0) {
        const int c = child_index(s);  // s is now the parent
        if (c < 3) {
            to_child(s, c + 1);
            return true;
        }
    }
    return false;
}

// The walk runs in the element's own frame (origin at the centroid, f1 and f2 in its plane,
// f3 its normal; built at upload): the field point is p = (p1, p2, p3), and a Gaussian point
// takes its offsets (da, db, dc) from the node coordinates in that frame.  The pair's local
// sums are rotated back once.  The frame of a sliver triangle is known only to eps times its
// aspect ratio, and the rounded centroid need not lie in the element's plane (a small element
// far from the origin: by a rounding of its coordinates), so the vertices keep their third
// coordinate in the frame (a rounding-level height) and a rectangle its corner relative to the
// centroid: with them the nodes are the exact combinations of the vertices, as in three
// dimensions.  A rectangle node's height varies across a cell only by rounding-level amounts
// (the sides' heights): the cell centre's height serves all its Gaussian points.
//
// Node geometry: a triangle node has a first vertex and two edge vectors (lattice position
// (i, j) in units of h = 2^-level along the root's edges B - A and C - A; an up node has
// vertices (i, j), (i+1, j), (i, j+1), a down node (i+1, j+1), (i, j+1), (i+1, j)); a
// rectangle node is the cell (i, j) of the h-grid along e1 and e2.
struct NearGeom {
    double ax, ay, az;  // triangle: root vertex A; rectangle: corner P0 (from the centroid)
    double ux, uy, uz;  // triangle: B - A; rectangle: e1 (in-plane, uz = 0)
    double vx, vy, vz;  // triangle: C - A; rectangle: e2 (in-plane, vz = 0)
};

// Node s: its first vertex (triangle) or centre (rectangle) and, for triangles, its edge
// vectors w1 = V1 - V0, w2 = V2 - V0; the node centroid c.
struct NodeGeom {
    double x0, y0, z0, w1x, w1y, w1z, w2x, w2y, w2z, cx, cy, cz;
};
__device__ __forceinline__ void node_geometry(const NearState& s, const NearGeom& g, double h, NodeGeom& n)
{
    if (s.kind == 0) {
        const double u = s.up ? s.i : s.i + 1, v = s.up ? s.j : s.j + 1, sg = s.up ? h : -h;
        n.x0 = fma(u * h, g.ux, fma(v * h, g.vx, g.ax));
        n.y0 = fma(u * h, g.uy, fma(v * h, g.vy, g.ay));
        n.z0 = fma(u * h, g.uz, fma(v * h, g.vz, g.az));
        n.w1x = sg * g.ux; n.w1y = sg * g.uy; n.w1z = sg * g.uz;
        n.w2x = sg * g.vx; n.w2y = sg * g.vy; n.w2z = sg * g.vz;
        n.cx = fma(1.0 / 3.0, n.w1x + n.w2x, n.x0);
        n.cy = fma(1.0 / 3.0, n.w1y + n.w2y, n.y0);
        n.cz = fma(1.0 / 3.0, n.w1z + n.w2z, n.z0);
    } else {
        const double ih = (s.i + 0.5) * h, jh = (s.j + 0.5) * h;
        n.cx = fma(ih, g.ux, fma(jh, g.vx, g.ax));
        n.cy = fma(ih, g.uy, fma(jh, g.vy, g.ay));
        n.cz = fma(ih, g.uz, fma(jh, g.vz, g.az));  // the height of the cell centre (rounding level)
        n.x0 = n.cx; n.y0 = n.cy; n.z0 = n.cz;
        n.w1x = n.w1y = n.w1z = n.w2x = n.w2y = n.w2z = 0.0;
    }
}

// Sums of one Gaussian point at offsets (da, db, dc) in the element's frame, weight w (unit
// element charge, without the factor near_scale):
//   field:        f0 += w/r, (f1, f2, f3) += w (da, db, dc)/r^3;
//   collocation:  f0 += w/r;
//   gradient:     f0 += w/r^3, (f1 .. f6) += w (da^2, db^2, dc^2, da db, da dc, db dc)/r^5.
template <int MODE>
constexpr bool near_potential() { return MODE == kNearColloc || MODE == kNearPhi; }
template <int MODE>
constexpr double near_scale()
{
    return near_potential<MODE>() ? HalfPower<1>::kappa
                               : (MODE == kNearEval ? HalfPower<3>::kappa : HalfPower<5>::kappa);
}
template <int MODE>
constexpr int near_sums() { return MODE == kNearGrad ? 7 : (near_potential<MODE>() ? 1 : 4); }
template <int MODE>
__device__ __forceinline__ void near_terms(double w, double da, double db, double dc, double (&f)[7])
{
    const double r2 = fma(da, da, fma(db, db, dc * dc));
    if constexpr (near_potential<MODE>()) {
        f[0] = add_inv_root(w, r2, f[0]);
    } else if constexpr (MODE == kNearEval) {
        const double w3 = inv_cube_phi(w, r2, f[0]);
        f[1] = fma(w3, da, f[1]);
        f[2] = fma(w3, db, f[2]);
        f[3] = fma(w3, dc, f[3]);
    } else {
        const double w5 = inv_fifth(w, r2);
        const double ua = w5 * da, ub = w5 * db, uc = w5 * dc;
        f[0] = fma(w5, r2, f[0]);  // w/r^3
        f[1] = fma(ua, da, f[1]);
        f[2] = fma(ub, db, f[2]);
        f[3] = fma(uc, dc, f[3]);
        f[4] = fma(ua, db, f[4]);
        f[5] = fma(ua, dc, f[5]);
        f[6] = fma(ub, dc, f[6]);
    }
}

// Pairs whose field point lies on the element (the trailing entries of the order, from
// *walk_end to the pair count): the exact integral about the point, one lane per pair; the
// walk kernel's lanes take them once the walks are done (grid-stride from `first`).  Per
// edge at distance h from the point with end offsets t1, t2 along it (rho^2 = h^2 + t^2):
// potential h [asinh(t/h)], field -n [(t/rho)(1 + ln rho) - asinh(t/h)] + h t [(1 + ln rho)/rho]
// (n the unit vector from the point's foot on the edge line towards the point's side).
template <int MODE>
__device__ __forceinline__ void on_element_pairs(const NearArgs& a, unsigned long long first, unsigned long long stride)
{
    constexpr bool COLLOC = MODE == kNearColloc;
    constexpr bool GRAD = MODE == kNearGrad;
    const Elements& el = a.el;
    const int64_t ne = el.ne;
    const unsigned long long total = min(a.ctr->near_count, a.near_cap);
    unsigned long long n_on = 0;
    for (unsigned long long w = *a.walk_end + first; w < total; w += stride) {
        const NearPair pr = a.opair[w];
        const unsigned long long cur = a.slot[a.order[w]];
        const int64_t e = pr.elem, p = pr.point;
        const bool tri = e < el.n_tri;
        double X[3];
        if (COLLOC) {
            X[0] = el.cen[p]; X[1] = el.cen[ne + p]; X[2] = el.cen[2 * ne + p];
        } else {
            X[0] = a.pts[p]; X[1] = a.pts[a.n + p]; X[2] = a.pts[2 * a.n + p];
        }
        double G[9], P[3], V[4][3];
        point_on_element(el, e, tri, X, G, P);  // (true: the cost pass put the pair here)
        const int nv = element_corners(el, e, tri, G, V);
        const double L = el.L[e];
        double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
        for (int k = 0; k < nv; ++k) {
            const double* Va = V[k];
            const double* Vb = V[(k + 1) % nv];
            double tv[3] = { Vb[0] - Va[0], Vb[1] - Va[1], Vb[2] - Va[2] };
            const double len = sqrt(tv[0] * tv[0] + tv[1] * tv[1] + tv[2] * tv[2]);
            tv[0] /= len; tv[1] /= len; tv[2] /= len;
            const double pa[3] = { Va[0] - P[0], Va[1] - P[1], Va[2] - P[2] };
            const double t1 = pa[0] * tv[0] + pa[1] * tv[1] + pa[2] * tv[2];
            const double t2 = t1 + len;
            double fn[3] = { pa[0] - t1 * tv[0], pa[1] - t1 * tv[1], pa[2] - t1 * tv[2] };
            const double hh = sqrt(fn[0] * fn[0] + fn[1] * fn[1] + fn[2] * fn[2]);
            if (!(hh > 1e-14 * L)) continue;
            fn[0] /= hh; fn[1] /= hh; fn[2] /= hh;
            const double r1 = sqrt(hh * hh + t1 * t1), r2 = sqrt(hh * hh + t2 * t2);
            const double as = asinh(t2 / hh) - asinh(t1 / hh);
            s0 += hh * as;
            const double l1 = 1.0 + log(r1), l2 = 1.0 + log(r2);
            const double gn = (t2 / r2) * l2 - (t1 / r1) * l1 - as;
            const double gt = hh * (l2 / r2 - l1 / r1);
            s1 += -gn * fn[0] + gt * tv[0];
            s2 += -gn * fn[1] + gt * tv[1];
            s3 += -gn * fn[2] + gt * tv[2];
        }
        const double inv_area = 1.0 / el.area[e];
        if (COLLOC) {
            a.res[cur] = s0 * inv_area;
        } else if (GRAD) {  // the normal field jumps across the element: no gradient there
            const double nan = __builtin_nan("");
            double2* r = reinterpret_cast<double2*>(a.res + 6 * cur);
            r[0] = make_double2(nan, nan);
            r[1] = make_double2(nan, nan);
            r[2] = make_double2(nan, nan);
        } else if (MODE == kNearPhi) {
            a.res[cur] = a.K * el.q[(int64_t)a.rhs * ne + e] * (s0 * inv_area);
        } else {
            const double Kq = a.K * el.q[(int64_t)a.rhs * ne + e];
            reinterpret_cast<double4*>(a.res)[cur] = make_double4(
                Kq * (s0 * inv_area), Kq * (s1 * inv_area), Kq * (s2 * inv_area), Kq * (s3 * inv_area));
        }
        n_on++;
    }
    if (n_on) atomicAdd(&a.ctr->on_surface, n_on);
}

// A list of at most this many pairs is walked a wavefront per pair, breadth first, whatever the pairs'
// depth: fewer than eleven pairs per resident wavefront, the lanes' walks would leave most of the
// chip idle.  Near stage so, and with the pairs that are not deep one per lane (3,600 elements, field):
// 16,500 pairs 0.41 and 0.63 ms, 34,600 pairs 0.28 and 0.50, 57,400 pairs 0.33 and 0.55, 107,000 pairs
// 0.39 and 0.58, 174,000 pairs 0.52 and 0.68 (gradient 0.64 and 0.72).  The line lies where the two were
// equal while a wavefront claimed its pairs one by one (40,000 pairs 0.71 and 0.55 ms); with several to a
// claim it is on the safe side: the wavefronts stay the faster to past 174,000 pairs.
constexpr unsigned long long kShortList = 32768;
constexpr unsigned kNearWindow = 64;  // entries of the order a wavefront claims at a time
constexpr unsigned long long kClaimMax = 8;  // deep pairs a wavefront claims at a time at most
constexpr int kNearWaves = kBlock / 64;
constexpr int kFront = 128;  // near nodes of one level of a breadth-first walk (per wavefront)
constexpr int kLeafQ = 128;  // leaves waiting for the rule: a batch of 64 and one chunk's more
constexpr unsigned kFrontUp = 1u << 31;  // orientation of a node in the near levels' stores

// One wavefront's share of LDS in the near kernel.
template <int NS>
struct NearLdsT {
    uint2 front[2][kFront];         // breadth-first walk: a level's near nodes, the next level's
    uint2 pos[kLeafQ];              // queued leaves
    uint16_t meta[kLeafQ];
    unsigned long long round[64];   // the lanes that queued a leaf, per round of a batch
    double res[NS][64];             // the batch's leaf sums
};

// A pair's walk set-up from the element's record: the element kind, its node geometry in the
// element's frame, the field point in that frame (offset from the centroid: numbers of the
// element's size, accurate for points very close to a small element far from the origin)
// and the threshold (near_dr L)^2.
template <int MODE>
__device__ __forceinline__ void pair_setup(const NearArgs& a, uint32_t p, uint32_t e, int& kind, NearGeom& g,
                                           double& p1, double& p2, double& p3, double& thr2)
{
    const Elements& el = a.el;
    const int64_t ne = el.ne;
    double P[3];
    if (MODE == kNearColloc) {
        P[0] = el.cen[p]; P[1] = el.cen[ne + p]; P[2] = el.cen[2 * ne + p];
    } else {
        P[0] = a.pts[p]; P[1] = a.pts[a.n + p]; P[2] = a.pts[2 * a.n + p];
    }
    kind = (int64_t)e < el.n_tri ? 0 : 1;
    double R[kNearRec];  // centroid, frame F, loc, thr2
    {
        const double2* rec = reinterpret_cast<const double2*>(el.nrec + (int64_t)e * kNearRec);
#pragma unroll
        for (int c = 0; c < 11; ++c) {
            const double2 v = rec[c];
            R[2 * c] = v.x;
            R[2 * c + 1] = v.y;
        }
    }
    const double* F = R + 3;
    const double* lc = R + 12;
    const double dxc = P[0] - R[0], dyc = P[1] - R[1], dzc = P[2] - R[2];
    p1 = fma(F[0], dxc, fma(F[1], dyc, F[2] * dzc));
    p2 = fma(F[3], dxc, fma(F[4], dyc, F[5] * dzc));
    p3 = fma(F[6], dxc, fma(F[7], dyc, F[8] * dzc));
    if (kind == 0) {  // vertices A', B', C' in the frame
        g.ax = lc[0]; g.ay = lc[1]; g.az = lc[6];
        g.ux = lc[2] - g.ax; g.uy = lc[3] - g.ay; g.uz = lc[7] - g.az;
        g.vx = lc[4] - g.ax; g.vy = lc[5] - g.ay; g.vz = lc[8] - g.az;
    } else {  // e1 = (2 gamma, 2 beta, h1), e2 = (2 alpha, 0, h2); the corner P0 - c
        g.ux = 2.0 * lc[0]; g.uy = 2.0 * lc[1]; g.uz = lc[6];
        g.vx = 2.0 * lc[2]; g.vy = 0.0; g.vz = lc[7];
        g.ax = lc[3]; g.ay = lc[4]; g.az = lc[5];
    }
    thr2 = R[21];
}

// The distance test of node s: its scale h = 2^-level, its geometry, and whether the point is
// within near_dr times the node's own L of its centroid.
__device__ __forceinline__ bool visit_node(const NearState& s, const NearGeom& g, double p1, double p2, double p3,
                                           double thr2, double& h, NodeGeom& nd)
{
    h = ldexp(1.0, -s.level);
    node_geometry(s, g, h, nd);
    const double qx = p1 - nd.cx, qy = p2 - nd.cy, qz = p3 - nd.cz;
    const double D2 = fma(qx, qx, fma(qy, qy, qz * qz));
    return D2 < thr2 * h * h;
}

// The element's rule on leaf node nd (scale h), weights scaled by the area ratio h^2, added to
// acc (the sums of near_terms in the element's frame); only the rule's nodes first, first + step, ...
template <int MODE>
__device__ __forceinline__ void leaf_add(int kind, const NearGeom& g, double p1, double p2, double p3,
                                         const NodeGeom& nd, double h, const double4* __restrict__ tri_nodes,
                                         const double4* __restrict__ rect_nodes, int nt, int nr, double (&acc)[7],
                                         int first = 0, int step = 1)
{
    double f[7] = { 0, 0, 0, 0, 0, 0, 0 };
    if (kind == 0) {
        const double q1 = p1 - nd.x0, q2 = p2 - nd.y0, q3 = p3 - nd.z0;
#pragma unroll 4
        for (int i = first; i < nt; i += step) {
            const double4 q = tri_nodes[i];
            const double lb = q.y, lc = q.z, w = q.w;
            const double da = fma(-lb, nd.w1x, fma(-lc, nd.w2x, q1));
            const double db = fma(-lb, nd.w1y, fma(-lc, nd.w2y, q2));
            const double dc = fma(-lb, nd.w1z, fma(-lc, nd.w2z, q3));
            near_terms<MODE>(w, da, db, dc, f);
        }
    } else {
        const double qx = p1 - nd.cx, qy = p2 - nd.cy, qz = p3 - nd.cz;
        const double H1x = h * (0.5 * g.ux), H1y = h * (0.5 * g.uy), H2x = h * (0.5 * g.vx);
#pragma unroll 4
        for (int i = first; i < nr; i += step) {
            const double4 q = rect_nodes[i];
            const double x = q.x, y = q.y, w = q.z;
            const double da = fma(-x, H1x, fma(-y, H2x, qx));
            const double db = fma(-x, H1y, qy);
            near_terms<MODE>(w, da, db, qz, f);
        }
    }
    const double h2 = near_scale<MODE>() * (h * h);
#pragma unroll
    for (int c = 0; c < near_sums<MODE>(); ++c) acc[c] = fma(h2, f[c], acc[c]);
}

// The pair's own result record at its slot (32 bytes for the field, 48 for the gradient);
// collocation keeps the unit-density potential (the densities are applied per right-hand
// side when the sums are formed).
template <int MODE>
__device__ __forceinline__ void write_record(const NearArgs& a, uint32_t e, unsigned long long cur,
                                             const double (&acc)[7])
{
    const Elements& el = a.el;
    if (MODE == kNearColloc) {
        a.res[cur] = acc[0];
        return;
    }
    const double Kq = a.K * el.q[(int64_t)a.rhs * el.ne + e];
    if (MODE == kNearPhi) {
        a.res[cur] = Kq * acc[0];
        return;
    }
    double F[9];
    {
        const double* rec = el.nrec + (int64_t)e * kNearRec + 3;
#pragma unroll
        for (int c = 0; c < 9; ++c) F[c] = rec[c];
    }
    if (MODE == kNearGrad) {
        // local tensor m = sum w d d^T / r^5 (d = (da, db, dc)), global M = F^T m F,
        // dE_i/dx_j = q (delta_ij S3 - 3 M_ij)
        const double m[3][3] = { { acc[1], acc[4], acc[5] },
                                 { acc[4], acc[2], acc[6] },
                                 { acc[5], acc[6], acc[3] } };
        double U[3][3];  // U[r][v] = sum_b m[r][b] F[b][v]
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int v = 0; v < 3; ++v) U[r][v] = fma(m[r][0], F[v], fma(m[r][1], F[3 + v], m[r][2] * F[6 + v]));
        auto M = [&](int u, int v) { return fma(F[u], U[0][v], fma(F[3 + u], U[1][v], F[6 + u] * U[2][v])); };
        double2* r = reinterpret_cast<double2*>(a.res + 6 * cur);
        r[0] = make_double2(Kq * fma(-3.0, M(0, 0), acc[0]), Kq * fma(-3.0, M(1, 1), acc[0]));
        r[1] = make_double2(Kq * fma(-3.0, M(2, 2), acc[0]), -3.0 * Kq * M(0, 1));
        r[2] = make_double2(-3.0 * Kq * M(0, 2), -3.0 * Kq * M(1, 2));
    } else {
        // local field sum w (da, db, dc)/r^3, rotated back
        reinterpret_cast<double4*>(a.res)[cur] = make_double4(
            Kq * acc[0], Kq * fma(F[0], acc[1], fma(F[3], acc[2], F[6] * acc[3])),
            Kq * fma(F[1], acc[1], fma(F[4], acc[2], F[7] * acc[3])),
            Kq * fma(F[2], acc[1], fma(F[5], acc[2], F[8] * acc[3])));
    }
}

// A node of a walk kept in LDS: its lattice position (i, j < 2^30), and a word with its level, its
// orientation and (one wavefront's queue of several pairs) the lane whose pair it belongs to.
__device__ __forceinline__ uint2 node_pos(const NearState& s) { return make_uint2((unsigned)s.i, (unsigned)s.j); }
__device__ __forceinline__ uint16_t node_meta(const NearState& s, int lane)
{
    return (uint16_t)(s.level | (s.up ? 32 : 0) | (lane << 6));
}
__device__ __forceinline__ NearState unpack_node(uint2 pos, unsigned meta, int kind)
{
    return NearState{ kind, (int)(meta & 31u), (int)pos.x, (int)pos.y, (meta & 32u) != 0 };
}

// Move to the next node of a depth-first walk of the subtree below `root` (level) after
// finishing node s; false when the walk has returned to the subtree's root.
__device__ __forceinline__ bool advance_within(NearState& s, int root)
{
    while (s.level > root) {
        const int c = child_index(s);  // s is now the parent
        if (c < 3) {
            to_child(s, c + 1);
            return true;
        }
    }
    return false;
}

// One lane walks the subtree below the near node s (above the depth cap) depth first and returns
// the nodes it visited.  It stops at its first leaf past `budget` visits, what the visit limit
// leaves of its pair's: a near limit of thousands has subtrees of billions of nodes.
template <int MODE>
__device__ int walk_subtree(NearState s, const NearGeom& g, double p1, double p2, double p3, double thr2,
                            int max_depth, int budget, const double4* __restrict__ tri_nodes,
                            const double4* __restrict__ rect_nodes, int nt, int nr, double (&acc)[7],
                            unsigned long long& n_leaves, unsigned long long& n_cap, int& max_level)
{
    const int root = s.level;
    int visits = 0;
    to_child(s, 0);
    while (true) {
        double h;
        NodeGeom nd;
        const bool near = visit_node(s, g, p1, p2, p3, thr2, h, nd);
        ++visits;
        if (s.level > max_level) max_level = s.level;
        if (near && s.level < max_depth && visits <= budget) {
            to_child(s, 0);
            continue;
        }
        leaf_add<MODE>(s.kind, g, p1, p2, p3, nd, h, tri_nodes, rect_nodes, nt, nr, acc);
        n_leaves++;
        if (near) n_cap++;
        if (visits > budget || !advance_within(s, root)) break;
    }
    return visits;
}

// A pair with a deep subdivision (the leading cost classes; every pair of a short list), walked by
// a whole wavefront breadth first: per level, the children of the level's near nodes are tested 64 at a time,
// the near ones (above the depth cap) form the next level, the others are leaves; leaves
// wait in LDS until 64 of them can take the rule loop together, one per lane.  A point very
// close to an element has a near region of some 65 nodes at every level (three node sizes
// around its foot), so its depth-first walk would take thousands of visits in one lane.
// Each lane sums its leaves in a fixed order; the lanes' sums are added by a fixed butterfly,
// so results are reproducible.  More near nodes in a level than kFront: the lane that found
// one walks its subtree depth first itself.  The visit limit ends the walk after the level, or
// after the single lanes' subtrees, with which the pair's visits pass it.
template <int MODE, typename NearLds>
__device__ void heavy_pair(const NearArgs& a, unsigned long long w, NearLds& q, const double4* __restrict__ tri_nodes, const double4* __restrict__ rect_nodes, int nt,
                           int nr, int lane, unsigned long long& n_leaves, unsigned long long& n_cap,
                           unsigned long long& n_limit, int& max_level)
{
    uint2* const leafq = q.pos;
    uint16_t* const leafm = q.meta;
    const NearPair pr = a.opair[w];
    const unsigned long long cur = a.slot[a.order[w]];
    int kind;
    NearGeom g;
    double p1, p2, p3, thr2;
    pair_setup<MODE>(a, pr.point, pr.elem, kind, g, p1, p2, p3, thr2);
    double acc[7] = { 0, 0, 0, 0, 0, 0, 0 };
    // the same in every lane: the current level's near nodes (nF, in cur_f: positions and
    // orientations), the next level's (nN), the next child of the level to test (base), the queued
    // leaves (nq), the visits
    uint2* cur_f = q.front[0];
    uint2* nxt_f = q.front[1];
    int level = 0;  // of the nodes in cur_f
    int nF = 1, nN = 0, base = 0, nq = 0;
    long long visits = 0;
    bool done = false;
    if (a.max_depth <= 0) {  // the rule on the element itself (depth cap 0): the root is the leaf
        if (lane == 0) {
            const NearState s{ kind, 0, 0, 0, true };
            double h;
            NodeGeom nd;
            n_leaves++;
            if (visit_node(s, g, p1, p2, p3, thr2, h, nd)) n_cap++;
            leafq[0] = node_pos(s);
            leafm[0] = node_meta(s, 0);
        }
        nq = 1;
        done = true;
    } else if (lane == 0) {
        cur_f[0] = make_uint2(kFrontUp, 0u);
    }
    wave_lds_sync();
    while (true) {
        if (!done && base >= 4 * nF) {  // the level is tested: on to the next one
            uint2* t = cur_f;
            cur_f = nxt_f;
            nxt_f = t;
            ++level;
            nF = nN;
            nN = 0;
            base = 0;
            if (nF == 0) {
                done = true;
            } else if (visits > a.visit_limit) {  // the limit ends the walk here
                if (lane == 0) n_limit++;
                done = true;
            }
        }
        if (nq >= 64 || (done && nq > 0)) {  // a batch of leaves, one per lane
            const int k = min(nq, 64);
            // fewer than 33 leaves: 2, 4, ... lanes to a leaf share its rule's nodes
            const int logk = k > 1 ? 32 - __builtin_clz((unsigned)(k - 1)) : 0;
            const int at = lane & ((1 << logk) - 1);
            if (at < k) {
                const NearState t = unpack_node(leafq[at], leafm[at], kind);
                double h;
                NodeGeom nd;
                (void)visit_node(t, g, p1, p2, p3, thr2, h, nd);
                leaf_add<MODE>(kind, g, p1, p2, p3, nd, h, tri_nodes, rect_nodes, nt, nr, acc, lane >> logk, 64 >> logk);
            }
            const uint2 rest = lane < nq - k ? leafq[k + lane] : make_uint2(0u, 0u);
            const uint16_t restm = lane < nq - k ? leafm[k + lane] : (uint16_t)0;
            wave_lds_sync();
            if (lane < nq - k) { leafq[lane] = rest; leafm[lane] = restm; }
            wave_lds_sync();
            nq -= k;
            continue;
        }
        if (done) break;
        // the next 64 children of the level's near nodes
        const int c = base + lane;
        const bool valid = c < 4 * nF;
        NearState s{ kind, 0, 0, 0, true };
        bool near = false;
        if (valid) {
            const uint2 f = cur_f[c >> 2];
            s = NearState{ kind, level, (int)(f.x & ~kFrontUp), (int)f.y, (f.x & kFrontUp) != 0 };
            to_child(s, c & 3);
            double h;
            NodeGeom nd;
            near = visit_node(s, g, p1, p2, p3, thr2, h, nd);
            if (s.level > max_level) max_level = s.level;
        }
        visits += (long long)__popcll(lane_mask(valid));
        const bool desc = valid && near && s.level < a.max_depth;
        const bool leaf = valid && !desc;
        if (leaf) {
            n_leaves++;
            if (near) n_cap++;
        }
        // descending children: the next level (index order); past kFront a lane walks its
        // child's subtree itself
        const unsigned long long dm = lane_mask(desc);
        const int pos = nN + (int)lanes_below(dm);
        const bool spill = desc && pos >= kFront;
        if (desc && !spill) nxt_f[pos] = make_uint2((unsigned)s.i | (s.up ? kFrontUp : 0u), (unsigned)s.j);
        nN = min(kFront, nN + (int)__popcll(dm));
        // leaves: the queue (fewer than 64 wait when a chunk adds at most 64)
        const unsigned long long lm = lane_mask(leaf);
        if (leaf) {
            leafq[nq + (int)lanes_below(lm)] = node_pos(s);
            leafm[nq + (int)lanes_below(lm)] = node_meta(s, 0);
        }
        nq += (int)__popcll(lm);
        base += 64;
        wave_lds_sync();
        if (lane_mask(spill) != 0ull) {
            int walked = 0;
            if (spill)
                walked = walk_subtree<MODE>(s, g, p1, p2, p3, thr2, a.max_depth, (int)(a.visit_limit - visits), tri_nodes,
                                            rect_nodes, nt, nr, acc, n_leaves, n_cap, max_level);
            for (int o = 32; o > 0; o >>= 1) walked += __shfl_xor(walked, o);  // (64 x 2^22 at most)
            visits += walked;
            if (visits > a.visit_limit) {
                if (lane == 0) n_limit++;
                done = true;
            }
        }
    }
    wave_lds_sync();  // the queue and the levels are reused by the next pair
    // the lanes' sums added by a fixed butterfly (every lane ends with the same total)
#pragma unroll
    for (int c = 0; c < near_sums<MODE>(); ++c)
        for (int o = 32; o > 0; o >>= 1) acc[c] += __shfl_xor(acc[c], o);
    if (lane == 0) write_record<MODE>(a, pr.elem, cur, acc);
}

// MODE: kNearEval (phi, E at field points), kNearColloc (phi at centroids, several density
// vectors), kNearGrad (field gradient at field points; NaN for a point on its element).
// The depth-first variant is held to four wavefronts per SIMD (128 registers): its workgroups
// then fit beside another stream's running far kernel (left alone the compiler takes 157).
// The field's other variant is held to three (left alone it takes 217 registers: two).
template <int MODE, bool DEEP>
__global__ __launch_bounds__(kBlock, !DEEP ? 4 : (MODE == kNearEval ? 3 : 1)) void near_kernel(NearArgs a)
{
    // the walks: the leading entries of the order (the points lying on their element follow);
    // the first `heavy` of them have deep subdivisions (DEEP: walked breadth first, a wavefront
    // each; else depth first like the others)
    const unsigned long long total = *a.walk_end;
    const unsigned long long heavy = !DEEP ? 0ull : (total <= kShortList ? total : (unsigned long long)*a.heavy_end);
    const int lane = lane_id();
    // the rules' nodes in LDS: a leaf's loop reads them at one address for the whole wavefront
    // (from global memory every node would be a vector load and a wait for it)
    extern __shared__ double4 near_rule_nodes[];  // [nt] triangle (la, lb, lc, w), [nr] rectangle (x, y, w, 0)
    __shared__ NearLdsT<near_sums<MODE>()> near_lds[kNearWaves];
    auto& Q = near_lds[threadIdx.x / 64];
    const int nt = a.rules.nt, nr = a.rules.nr;
    // Every wavefront's first deep pair and first window are its own by its index; the shared
    // cursors hand out what follows.  (Claiming those too, a launch's four thousand wavefronts
    // queue up at one address: 102 shallow pairs took 75 us, 16 us so.)
    const unsigned long long waves = (unsigned long long)gridDim.x * kNearWaves;
    const unsigned long long wave = (unsigned long long)blockIdx.x * kNearWaves + threadIdx.x / 64;
    const unsigned long long first_wave = (unsigned long long)blockIdx.x * kNearWaves;
    if (first_wave < heavy || heavy + first_wave * kNearWindow < total) {  // the workgroup has walks
        for (int i = threadIdx.x; i < nt + nr; i += kBlock) {
            const double* src = i < nt ? a.rules.tri + 4 * i : a.rules.rect + 4 * (i - nt);
            near_rule_nodes[i] = make_double4(src[0], src[1], src[2], src[3]);
        }
        __syncthreads();
    }
    const double4* __restrict__ tri_nodes = near_rule_nodes;
    const double4* __restrict__ rect_nodes = near_rule_nodes + nt;

    unsigned long long n_leaves = 0, n_cap = 0, n_limit = 0;
    int max_level = 0;

    // ---- the deep pairs, one per wavefront at a time
    if (DEEP) {
        // (a claim takes more of them the longer the list: at one address about 80 claims are served in
        // a microsecond, and one by one 26,000 pairs' claims took longer than their walks - near stage
        // 0.54 ms, 0.28 ms so; 16 at most instead of 8 leave the last wavefronts too far behind, 0.25
        // ms against 0.23 at 28,000 pairs)
        const unsigned long long claim = min(max(heavy / waves, 1ull), kClaimMax);
        for (unsigned long long hw = wave, end = wave + 1; hw < heavy;) {
            heavy_pair<MODE>(a, hw, Q, tri_nodes, rect_nodes, nt, nr, lane, n_leaves, n_cap, n_limit, max_level);
            if (++hw < end) continue;
            if (heavy <= waves) break;
            if (lane == 0) hw = waves + atomicAdd(&a.ctr->heavy_cursor, claim);
            hw = bcast_u64(hw, 0);
            end = hw + claim;
        }
    }

    // ---- the other pairs, 64 at a time: each lane walks one depth first, but only down to its
    // leaves, which it queues; 64 queued leaves then take the rule together, one per lane,
    // whichever pairs they come from.  A leaf's rule costs about fifteen times the steps that find
    // it, so a wavefront with one long walk left still works on all lanes (with the rule in the
    // walk's own loop such walks, hundreds of leaves long, set the kernel's time).  Each pair's
    // lane adds its leaves one after another in the order of its walk, so the sum does not depend on
    // which other pairs share the wavefront.
    enum { kIdle = 0, kWalking = 1, kWalked = 2, kOut = 3 };
    int state = kIdle;
    bool found = false, is_near = false;  // the walk stands at a leaf that is not queued yet
    NearState st{ 0, 0, 0, 0, true };
    uint32_t e = 0;
    unsigned long long cur = 0;  // result slot of the pair in hand
    NearGeom g{};
    double p1 = 0.0, p2 = 0.0, p3 = 0.0;  // the field point in the element's frame
    double thr2 = 0.0, acc[7] = { 0, 0, 0, 0, 0, 0, 0 };
    int64_t visits = 0;
    // the wavefront's window of the order (the same in every lane): kNearWindow consecutive
    // entries claimed with one atomic, handed to its lanes as they need pairs; consecutive
    // entries are pairs of one cost class, so the lanes walk trees of one kind and similar size
    unsigned long long win = heavy + wave * kNearWindow, win_end = win + kNearWindow;

    const bool more = heavy + waves * kNearWindow < total;  // windows beyond the first ones
    for (bool go = win < total; go;) {
        // ---- refill from the window (a new window when it is used up)
        const unsigned long long need = lane_mask(state == kIdle);
        if (need) {
            if (win >= win_end) {
                win = total;
                if (more) {
                    const int first = __ffsll((long long)need) - 1;
                    unsigned long long b = 0;
                    if (lane == first) b = atomicAdd(&a.ctr->cursor, (unsigned long long)kNearWindow);
                    win = heavy + waves * kNearWindow + bcast_u64(b, first);
                }
                win_end = win + kNearWindow;
            }
            const unsigned rank = lanes_below(need);
            const unsigned long long avail = win_end - win, w = win + rank;
            win += min(avail, (unsigned long long)__popcll(need));
            // a lane without an entry (the window ran out) waits for the next one
            if (state == kIdle && rank < avail) {
                if (w >= total) {
                    state = kOut;
                } else {
                    const NearPair pr = a.opair[w];  // most expensive pairs first
                    cur = a.slot[a.order[w]];
                    e = pr.elem;
                    pair_setup<MODE>(a, pr.point, pr.elem, st.kind, g, p1, p2, p3, thr2);
#pragma unroll
                    for (int c = 0; c < 7; ++c) acc[c] = 0.0;
                    visits = 0;
                    state = kWalking;
                    found = false;
                    st.i = 0; st.j = 0; st.up = true;
                    if (a.max_depth <= 0) st.level = 0;  // evaluate the rule on the element itself (depth cap)
                    else st.level = 1;                   // first child of the root
                }
            }
        }
        // ---- queue leaves in rounds, at most one per lane and round
        int nq = 0, rounds = 0;
        while (nq < 64) {
            const bool walking = state == kWalking;
            const unsigned long long wm = lane_mask(walking);
            if (wm == 0ull) break;
            if (walking && !found) {  // from st down to the next leaf
                double h;
                NodeGeom nd;
                while (true) {
                    is_near = visit_node(st, g, p1, p2, p3, thr2, h, nd);
                    ++visits;
                    if (st.level > max_level) max_level = st.level;
                    if (!(is_near && st.level < a.max_depth && visits <= a.visit_limit)) break;
                    to_child(st, 0);
                }
                found = true;
            }
            const int pos = nq + (int)lanes_below(wm);
            const bool take = walking && pos < 64;
            const unsigned long long tm = lane_mask(take);
            if (lane == 0) Q.round[rounds] = tm;
            ++rounds;
            nq += (int)__popcll(tm);
            if (take) {
                Q.pos[pos] = node_pos(st);
                Q.meta[pos] = node_meta(st, lane);
                found = false;
                n_leaves++;
                if (is_near) n_cap++;
                if (visits > a.visit_limit) {
                    n_limit++;
                    state = kWalked;
                } else if (!advance(st)) {
                    state = kWalked;
                }
            }
        }
        if (nq == 0) {
            go = lane_mask(state != kOut) != 0ull;
            continue;
        }
        wave_lds_sync();
        // ---- the rule on the queued leaves, one per lane, with their pairs' geometry
        {
            const int at = min(lane, nq - 1);
            const uint2 lp = Q.pos[at];
            const unsigned lm = Q.meta[at];
            const int o = (int)(lm >> 6);
            NearGeom og;
            og.ax = __shfl(g.ax, o); og.ay = __shfl(g.ay, o); og.az = __shfl(g.az, o);
            og.ux = __shfl(g.ux, o); og.uy = __shfl(g.uy, o); og.uz = __shfl(g.uz, o);
            og.vx = __shfl(g.vx, o); og.vy = __shfl(g.vy, o); og.vz = __shfl(g.vz, o);
            const double o1 = __shfl(p1, o), o2 = __shfl(p2, o), o3 = __shfl(p3, o);
            const NearState t = unpack_node(lp, lm, __shfl(st.kind, o));
            if (lane < nq) {
                const double h = ldexp(1.0, -t.level);
                NodeGeom nd;
                node_geometry(t, og, h, nd);
                double f[7] = { 0, 0, 0, 0, 0, 0, 0 };
                leaf_add<MODE>(t.kind, og, o1, o2, o3, nd, h, tri_nodes, rect_nodes, nt, nr, f);
#pragma unroll
                for (int c = 0; c < near_sums<MODE>(); ++c) Q.res[c][lane] = f[c];
            }
        }
        wave_lds_sync();
        // ---- each pair's lane adds its leaves in the order of its walk
        for (int r = 0, first = 0; r < rounds; ++r) {
            const unsigned long long tm = Q.round[r];
            if ((tm >> lane) & 1ull) {
                const int at = first + (int)lanes_below(tm);
#pragma unroll
                for (int c = 0; c < near_sums<MODE>(); ++c) acc[c] += Q.res[c][at];
            }
            first += (int)__popcll(tm);
        }
        if (state == kWalked) {
            write_record<MODE>(a, e, cur, acc);
            state = kIdle;
        }
        wave_lds_sync();  // the queue is filled again
    }

    // the lanes' counters, added up over the workgroup: one atomic per counter and workgroup (one per
    // lane took longer than the walks of a short list: 262,000 of them at one address)
    {
        __shared__ unsigned long long total_of[4];
        if (threadIdx.x < 4) total_of[threadIdx.x] = 0ull;
        for (int o = 32; o > 0; o >>= 1) {
            n_leaves += __shfl_xor(n_leaves, o);
            n_cap += __shfl_xor(n_cap, o);
            n_limit += __shfl_xor(n_limit, o);
            max_level = max(max_level, __shfl_xor(max_level, o));
        }
        __syncthreads();
        if (lane == 0 && n_leaves) {
            atomicAdd(&total_of[0], n_leaves);
            if (n_cap) atomicAdd(&total_of[1], n_cap);
            if (n_limit) atomicAdd(&total_of[2], n_limit);
            atomicMax(&total_of[3], (unsigned long long)max_level);
        }
        __syncthreads();
        if (threadIdx.x == 0 && total_of[0]) {
            atomicAdd(&a.ctr->leaves, total_of[0]);
            if (total_of[1]) atomicAdd(&a.ctr->cap_hits, total_of[1]);
            if (total_of[2]) atomicAdd(&a.ctr->visit_limit_hits, total_of[2]);
            if (total_of[3]) atomicMax(&a.ctr->max_depth, total_of[3]);
        }
    }

    // then the pairs whose point lies on the element (after the walk loop: none of its
    // state is live here, so the closed form does not add to the walk's registers)
    on_element_pairs<MODE>(a, (unsigned long long)blockIdx.x * kBlock + threadIdx.x,
                           (unsigned long long)gridDim.x * kBlock);
}

// ---------------------------------------------------------------- small kernels -----
// One 192-byte record per element with what the near walk reads when it takes a pair (three
// 64-byte lines instead of 22 from the separate arrays): centroid, frame, loc, thr2.
__global__ void pack_near_records_kernel(Elements el, double* __restrict__ nrec)
{
    const int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t ne = el.ne;
    if (e >= ne) return;
    double r[kNearRec];
#pragma unroll
    for (int c = 0; c < 3; ++c) r[c] = el.cen[c * ne + e];
#pragma unroll
    for (int c = 0; c < 9; ++c) r[3 + c] = el.frame[c * ne + e];
#pragma unroll
    for (int c = 0; c < 9; ++c) r[12 + c] = el.loc[c * ne + e];
    r[21] = el.thr2[e];
    r[22] = 0.0;
    r[23] = 0.0;
    double2* out = reinterpret_cast<double2*>(nrec + e * kNearRec);
#pragma unroll
    for (int c = 0; c < kNearRec / 2; ++c) out[c] = make_double2(r[2 * c], r[2 * c + 1]);
}

__global__ void charges_kernel(const double* sigma, const double* area, double* q, int64_t ne, int n_rhs)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= ne * n_rhs) return;
    q[i] = sigma[i] * area[i % ne];
}

__global__ void zero_counters_kernel(DevCounters* c)
{
    unsigned long long* w = reinterpret_cast<unsigned long long*>(c);
    const int i = threadIdx.x;
    if (i < (int)(sizeof(DevCounters) / sizeof(unsigned long long))) w[i] = 0ull;
}

// LDS of a workgroup from which four, not five, fit a CU (160 KB), and leave 30 KB
constexpr size_t kBesideLds = 33280;

template <bool DR, int NT, int NR, int T1, int T2, int T3, int R1, int R2, int R3, bool MIXED, int PPT, int MODE>
hipError_t far_eval_launch(const FarArgs& a, hipStream_t s)
{
    // Batches of other streams run beside a served one: five workgroups of the mixed kernel with one point per
    // lane (90 registers) would leave a CU 32 registers per lane, and the list pass (62 or 87) and the near
    // kernel (120) of a short batch would wait for its workgroups to end, each some milliseconds
    // long; four leave 128 (120 queries, 1,000,000 elements: p50 91 ms with five, 31 with four).
    // The distance-ratio kernel with two points per lane (119 registers, four workgroups) gets no spare
    // LDS: two workgroups a CU instead cost more than the short queries gain (40 queries/s, 1,000,000
    // elements: short p50 25 -> 8 ms, but saturation 52 -> 37 queries/s and p99 0.54 -> 1.82 s).
    using Tile = TileLds<MIXED, 1, !MIXED && PPT == 1 && MODE != kFarGrad>;
    const size_t spare = a.beside && MIXED && PPT == 1 && sizeof(Tile) < kBesideLds ? kBesideLds - sizeof(Tile) : 0;
    const int64_t per = (int64_t)kBlock * PPT;
    const int64_t blocks = (a.n + per - 1) / per;
    if (blocks > 0x7fffffff || a.n_split < 1 || a.n_split > 65535) return hipErrorInvalidValue;
    far_eval_kernel<DR, NT, NR, T1, T2, T3, R1, R2, R3, MIXED, PPT, MODE>
        <<<dim3((unsigned)blocks, (unsigned)a.n_split), dim3(kBlock), spare, s>>>(a);
    return hipGetLastError();
}

// Points up to which a lane takes one: a workgroup of three per lane would be partly empty (256 points x
// 150,000 elements, FP64 far kernel 2.13 ms, 0.78 ms with one; by distance ratio 1.42 and 0.76 ms).
constexpr int64_t kOnePoint = 2048;

// Field points per lane: two for the distance-ratio levels and the run-time rules; for the
// compiled long rules three in FP64 and one in the mixed path (on the 150k-element cylinder
// 1 % and 2 % faster than two; four was slower in both).
template <bool MIXED>
hipError_t far_eval_dispatch(const FarArgs& a, hipStream_t s)
{
    constexpr int PPT = 2;
    constexpr int PPT_LONG = MIXED ? 1 : 3;
    if (a.dr_rules) {
        const int* t = a.lv.tri_off;
        const int* r = a.lv.rect_off;
        const bool std_levels = t[1] == 7 && t[2] == 19 && t[3] == 38 && r[1] == 7 && r[2] == 19 && r[3] == 36;
        if (std_levels && t[4] - t[3] == 33 && r[4] - r[3] == 49)
            return a.n <= kOnePoint ? far_eval_launch<true, 7, 7, 12, 19, 33, 12, 17, 49, MIXED, 1, kFarField>(a, s)
                                    : far_eval_launch<true, 7, 7, 12, 19, 33, 12, 17, 49, MIXED, PPT, kFarField>(a, s);
        return far_eval_launch<true, 0, 0, 0, 0, 0, 0, 0, 0, MIXED, PPT, kFarField>(a, s);
    }
    const int nt = a.rules.nt, nr = a.rules.nr;
    // a small evaluation (fewer than 1024 workgroups at three points per lane: under one
    // wavefront per SIMD and four per CU) takes one point per lane: more wavefronts hide the
    // latency of the dependent FP64 chains
    const bool small = !MIXED && (a.n <= kOnePoint || (a.n + 3 * kBlock - 1) / (3 * kBlock) * a.n_split < 1024);
    if (small && nr == 49 && nt == 7) return far_eval_launch<false, 7, 49, 0, 0, 0, 0, 0, 0, MIXED, 1, kFarField>(a, s);
    if (small && nr == 49 && nt == 33) return far_eval_launch<false, 33, 49, 0, 0, 0, 0, 0, 0, MIXED, 1, kFarField>(a, s);
    if (nr == 49) {
        if (nt == 7) return far_eval_launch<false, 7, 49, 0, 0, 0, 0, 0, 0, MIXED, PPT_LONG, kFarField>(a, s);
        if (nt == 12) return far_eval_launch<false, 12, 49, 0, 0, 0, 0, 0, 0, MIXED, PPT_LONG, kFarField>(a, s);
        if (nt == 19) return far_eval_launch<false, 19, 49, 0, 0, 0, 0, 0, 0, MIXED, PPT_LONG, kFarField>(a, s);
        if (nt == 33) return far_eval_launch<false, 33, 49, 0, 0, 0, 0, 0, 0, MIXED, PPT_LONG, kFarField>(a, s);
    }
    if (nr == 33 && nt == 33)  // Table B5 for the rectangles
        return far_eval_launch<false, 33, 33, 0, 0, 0, 0, 0, 0, MIXED, PPT_LONG, kFarField>(a, s);
    return far_eval_launch<false, 0, 0, 0, 0, 0, 0, 0, 0, MIXED, PPT, kFarField>(a, s);
}

// Potential alone: compiled for the default rules, the 7-point triangle rule and the levels.  FP64: 7
// instead of 12 FP64 instructions per node beside the reciprocal square root, mixed 5 instead of 9, and
// no rotation back (131,071 points x 150,000 elements by distance ratio, mixed: far kernel 85.0 -> 52.6 ms).
// Other rules take the run-time kernel, which is still faster than the field's compiled ones (20,000 points x
// 18,000 elements: 33-point / Table B5 4.7 and 6.4 ms, 12-point / 7 x 7 4.0 and 5.3; mixed 2.0 and 3.4, 1.8 and 2.5).
template <bool MIXED>
hipError_t far_phi_dispatch(const FarArgs& a, hipStream_t s)
{
    constexpr int PPT = 2;
    constexpr int PPT_LONG = MIXED ? 2 : 3;
    const bool one = a.n <= kOnePoint;
    if (a.dr_rules) {
        const int* t = a.lv.tri_off;
        const int* r = a.lv.rect_off;
        const bool std_levels = t[1] == 7 && t[2] == 19 && t[3] == 38 && r[1] == 7 && r[2] == 19 && r[3] == 36;
        if (std_levels && t[4] - t[3] == 33 && r[4] - r[3] == 49)
            return one ? far_eval_launch<true, 7, 7, 12, 19, 33, 12, 17, 49, MIXED, 1, kFarPhi>(a, s)
                       : far_eval_launch<true, 7, 7, 12, 19, 33, 12, 17, 49, MIXED, PPT, kFarPhi>(a, s);
        return far_eval_launch<true, 0, 0, 0, 0, 0, 0, 0, 0, MIXED, PPT, kFarPhi>(a, s);
    }
    const int nt = a.rules.nt, nr = a.rules.nr;
    if (nr == 49 && nt == 33)
        return one ? far_eval_launch<false, 33, 49, 0, 0, 0, 0, 0, 0, MIXED, 1, kFarPhi>(a, s)
                   : far_eval_launch<false, 33, 49, 0, 0, 0, 0, 0, 0, MIXED, PPT_LONG, kFarPhi>(a, s);
    if (nr == 49 && nt == 7)
        return one ? far_eval_launch<false, 7, 49, 0, 0, 0, 0, 0, 0, MIXED, 1, kFarPhi>(a, s)
                   : far_eval_launch<false, 7, 49, 0, 0, 0, 0, 0, 0, MIXED, PPT_LONG, kFarPhi>(a, s);
    return far_eval_launch<false, 0, 0, 0, 0, 0, 0, 0, 0, MIXED, PPT, kFarPhi>(a, s);
}

// Gradient: compile-time node counts for the default rules only; one point per lane for
// those (FP64, 15,000 points x 150,000 elements: far kernel 53.9 ms, 56.6 ms with two; mixed the
// same with one and two), two with the levels (52.3 ms, 53.3 ms with one).
template <bool MIXED>
hipError_t far_grad_dispatch(const FarArgs& a, hipStream_t s)
{
    constexpr int PPT = 2;
    constexpr int PPT_LONG = 1;
    if (a.dr_rules) {
        const int* t = a.lv.tri_off;
        const int* r = a.lv.rect_off;
        const bool std_levels = t[1] == 7 && t[2] == 19 && t[3] == 38 && r[1] == 7 && r[2] == 19 && r[3] == 36;
        if (std_levels && t[4] - t[3] == 33 && r[4] - r[3] == 49)
            return far_eval_launch<true, 7, 7, 12, 19, 33, 12, 17, 49, MIXED, PPT, kFarGrad>(a, s);
        return far_eval_launch<true, 0, 0, 0, 0, 0, 0, 0, 0, MIXED, PPT, kFarGrad>(a, s);
    }
    if (a.rules.nt == 33 && a.rules.nr == 49)
        return far_eval_launch<false, 33, 49, 0, 0, 0, 0, 0, 0, MIXED, PPT_LONG, kFarGrad>(a, s);
    return far_eval_launch<false, 0, 0, 0, 0, 0, 0, 0, 0, MIXED, PPT, kFarGrad>(a, s);
}

template <int NT, int NR, bool MIXED, int PPT>
hipError_t far_colloc_launch(const FarArgs& a, hipStream_t s)
{
    const int64_t per = (int64_t)kBlock * PPT;
    const int64_t blocks = (a.el.ne + per - 1) / per;
    if (blocks > 0x7fffffff || a.n_split < 1 || a.n_split > 65535) return hipErrorInvalidValue;
    far_colloc_kernel<NT, NR, MIXED, PPT><<<dim3((unsigned)blocks, (unsigned)a.n_split), dim3(kBlock), 0, s>>>(a);
    return hipGetLastError();
}

// Collocation points per lane: three in FP64, two in the mixed path (on the 200,000-element
// nested cylinders 1.5 % faster than two in FP64; one was slower in both, three slower mixed).
template <bool MIXED>
hipError_t far_colloc_dispatch(const FarArgs& a, hipStream_t s)
{
    constexpr int PPT = MIXED ? 2 : 3;
    if (a.rules.nr == 49 && a.rules.nt == 33) {
        // few workgroups at PPT points per lane: one point (FP64, 2,976 elements 208 -> 165 us, 8,000 elements
        // 1.05 -> 0.91 ms; mixed 111 -> 96 us and 0.42 -> 0.47 ms, where the node reads bound it)
        if ((a.el.ne + PPT * kBlock - 1) / (PPT * kBlock) * a.n_split < (MIXED ? 768 : 2048)) return far_colloc_launch<33, 49, MIXED, 1>(a, s);
        return far_colloc_launch<33, 49, MIXED, PPT>(a, s);
    }
    return far_colloc_launch<0, 0, MIXED, PPT>(a, s);
}

}  // namespace

hipError_t launch_far_eval(const FarArgs& a, int precision, hipStream_t s)
{
    if (a.n <= 0) return hipSuccess;
    if (a.n_out == 1) return precision == 1 ? far_phi_dispatch<true>(a, s) : far_phi_dispatch<false>(a, s);
    return precision == 1 ? far_eval_dispatch<true>(a, s) : far_eval_dispatch<false>(a, s);
}

namespace {
template <bool DR, int MODE>
hipError_t far_few_launch(const FarArgs& a, hipStream_t s)
{
    const RuleTables& R = DR ? a.lv.tab : a.rules;
    const size_t lds = (size_t)(R.nt + R.nr) * sizeof(double4);
    if (a.n <= 2)
        far_few_kernel<DR, 1, MODE><<<dim3((unsigned)a.n_split, (unsigned)a.n), kBlock, lds, s>>>(a);
    else
        far_few_kernel<DR, 4, MODE><<<dim3((unsigned)a.n_split, (unsigned)((a.n + 3) / 4)), kBlock, lds, s>>>(a);
    return hipGetLastError();
}
}  // namespace

// Few points (at most kFewPoints): chunk partial sums, and the near pairs to the list.
hipError_t launch_far_few(const FarArgs& a, int mode, hipStream_t s)
{
    if (a.n <= 0 || a.n > kFewPoints || !a.partial || a.n_split < 1 || a.n_split > 65535 ||
        a.chunk * a.n_split < a.el.ne)
        return hipErrorInvalidValue;
    if (mode == kNearGrad) return a.dr_rules ? far_few_launch<true, kFarGrad>(a, s) : far_few_launch<false, kFarGrad>(a, s);
    if (a.n_out == 1) return a.dr_rules ? far_few_launch<true, kFarPhi>(a, s) : far_few_launch<false, kFarPhi>(a, s);
    return a.dr_rules ? far_few_launch<true, kFarField>(a, s) : far_few_launch<false, kFarField>(a, s);
}

hipError_t launch_far_colloc(const FarArgs& a, int precision, hipStream_t s)
{
    if (a.el.ne <= 0) return hipSuccess;
    return precision == 1 ? far_colloc_dispatch<true>(a, s) : far_colloc_dispatch<false>(a, s);
}

hipError_t launch_far_grad(const FarArgs& a, int precision, hipStream_t s)
{
    if (a.n <= 0) return hipSuccess;
    return precision == 1 ? far_grad_dispatch<true>(a, s) : far_grad_dispatch<false>(a, s);
}

// Workgroups of a persistent near kernel: as many as the GPU holds at once (a workgroup beyond
// them would start its own first pairs, the expensive ones, when the others are through), no more
// than the list can hold pairs.  Every lane leaves once the pairs are handed out.
template <int MODE, bool DEEP>
static hipError_t launch_near_kernel(const NearArgs& a, hipStream_t s)
{
    const size_t lds = (size_t)(a.rules.nt + a.rules.nr) * sizeof(double4);
    // a fact of the kernel and the GPU (gfx950 alone), asked for once: with the largest rules' LDS
    static const unsigned long long most = [] {
        int dev = 0, cus = 0, per_cu = 0;
        const size_t largest = (size_t)(kMaxTriNodes + kMaxRectNodes) * sizeof(double4);
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, near_kernel<MODE, DEEP>, kBlock, largest) != hipSuccess)
            (void)hipGetLastError();
        return (unsigned long long)std::max(1, cus * std::max(1, per_cu));
    }();
    const unsigned blocks = (unsigned)std::max<unsigned long long>(1, std::min(most, (a.near_cap + kNearWaves - 1) / kNearWaves));
    near_kernel<MODE, DEEP><<<blocks, kBlock, lds, s>>>(a);
    return hipGetLastError();
}

hipError_t launch_near(const NearArgs& a, int mode, hipStream_t s)
{
    if (mode == kNearColloc) return launch_near_kernel<kNearColloc, true>(a, s);
    if (mode == kNearGrad) return launch_near_kernel<kNearGrad, true>(a, s);
    if (mode == kNearPhi) return launch_near_kernel<kNearPhi, true>(a, s);
    return a.deep ? launch_near_kernel<kNearEval, true>(a, s) : launch_near_kernel<kNearEval, false>(a, s);
}

hipError_t launch_near_list(const double* pts, int64_t n, const Elements& el, NearPair* list, unsigned long long cap,
                            DevCounters* ctr, hipStream_t s)
{
    if (n <= 0 || el.ne <= 0) return hipSuccess;
    const int64_t blocks = (n + kListPoints - 1) / kListPoints;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    // few point blocks (a small evaluation): split the elements into chunks (multiples of 16
    // elements), up to about 2048 workgroups in all
    const int64_t units = (el.ne + 15) / 16;
    const int64_t split = std::max<int64_t>(1, std::min<int64_t>({ (2048 + blocks - 1) / blocks, units, 65535 }));
    const int64_t chunk = ((units + split - 1) / split) * 16;
    const int64_t chunks = (el.ne + chunk - 1) / chunk;
    const dim3 grid((unsigned)blocks, (unsigned)chunks);
    if (chunk > kListFine) near_list_kernel<true><<<grid, kBlock, 0, s>>>(pts, n, el, list, cap, ctr, chunk);
    else near_list_kernel<false><<<grid, kBlock, 0, s>>>(pts, n, el, list, cap, ctr, chunk);
    return hipGetLastError();
}

hipError_t launch_pack_near_records(const Elements& el, double* nrec, hipStream_t s)
{
    if (el.ne <= 0) return hipSuccess;
    pack_near_records_kernel<<<(unsigned)((el.ne + kBlock - 1) / kBlock), kBlock, 0, s>>>(el, nrec);
    return hipGetLastError();
}

hipError_t launch_charges(const double* sigma, const double* area, double* q, int64_t ne, int n_rhs, hipStream_t s)
{
    const int64_t tot = ne * n_rhs;
    if (tot <= 0) return hipSuccess;
    charges_kernel<<<(unsigned)((tot + 255) / 256), 256, 0, s>>>(sigma, area, q, ne, n_rhs);
    return hipGetLastError();
}

// ------------------------------------------------------------ solver support -------
// Potential of an element with unit density at its own centroid, K times the exact polar
// integral (per edge at distance h with end offsets t1, t2: h [asinh(t2/h) - asinh(t1/h)]):
// the diagonal of the collocation matrix.
__global__ void self_diag_kernel(Elements el, double K, double* __restrict__ diag)
{
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t ne = el.ne;
    if (e >= ne) return;
    double G[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) G[c] = el.geom[(int64_t)c * ne + e];
    double V[4][3];
    int nv;
    if (e < el.n_tri) {
        nv = 3;
#pragma unroll
        for (int c = 0; c < 3; ++c) { V[0][c] = 0.0; V[1][c] = G[3 + c] - G[c]; V[2][c] = G[6 + c] - G[c]; V[3][c] = 0.0; }
    } else {
        nv = 4;
#pragma unroll
        for (int c = 0; c < 3; ++c) { V[0][c] = 0.0; V[1][c] = G[3 + c]; V[2][c] = G[3 + c] + G[6 + c]; V[3][c] = G[6 + c]; }
    }
    double P[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) P[c] = el.cen[c * ne + e] - G[c];
    double sum = 0.0;
    for (int k = 0; k < nv; ++k) {
        const double* Va = V[k];
        const double* Vb = V[(k + 1) % nv];
        double tv[3] = { Vb[0] - Va[0], Vb[1] - Va[1], Vb[2] - Va[2] };
        const double len = sqrt(tv[0] * tv[0] + tv[1] * tv[1] + tv[2] * tv[2]);
        tv[0] /= len; tv[1] /= len; tv[2] /= len;
        const double pa[3] = { Va[0] - P[0], Va[1] - P[1], Va[2] - P[2] };
        const double t1 = pa[0] * tv[0] + pa[1] * tv[1] + pa[2] * tv[2];
        const double fx = pa[0] - t1 * tv[0], fy = pa[1] - t1 * tv[1], fz = pa[2] - t1 * tv[2];
        const double h = sqrt(fx * fx + fy * fy + fz * fz);
        if (h > 0.0) sum += h * (asinh((t1 + len) / h) - asinh(t1 / h));
    }
    diag[e] = K * sum;
}

// partial[j][b] = sum over block b's share of V[j][i] * w[i] (fixed order); blockIdx.y = j < k: the vectors
// side by side (one after the other in a workgroup, each waited for the last one's reduction)
__global__ void multi_dot_kernel(const double* __restrict__ V, int64_t n, const double* __restrict__ w,
                                 double* __restrict__ partial)
{
    __shared__ double red[4];
    const int j = blockIdx.y;
    double acc = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        acc = fma(V[(int64_t)j * n + i], w[i], acc);
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
    if (lane_id() == 0) red[threadIdx.x / 64] = acc;
    __syncthreads();
    if (threadIdx.x == 0) partial[(int64_t)j * gridDim.x + blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// y[i] = a * y[i] + sum_j c[j] V[j][i] / d[i]^p  (p = 0 or 1; d may be null when p = 0)
// The coefficients come with the launch: no copy to wait for.
__global__ void combine_kernel(double* __restrict__ y, double a, const double* __restrict__ V, CombineCoef c, int k,
                               int64_t n, const double* __restrict__ d)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
#pragma unroll 4
    for (int j = 0; j < k; ++j) s = fma(c.c[j], V[(int64_t)j * n + i], s);
    if (d) s /= d[i];
    y[i] = a == 0.0 ? s : fma(a, y[i], s);  // (a = 0: y need not hold numbers yet)
}

// h[j] = sum over b of partial[j][b] (in that order), y -= sum_j h[j] V[j]: a Gram-Schmidt pass whose
// coefficients need not go through the host (a copy, a wait and a launch that finds the GPU idle, about
// 25 us between two products of 165 us).  Every workgroup forms all h, a thread each; k <= 256.
__global__ void project_kernel(double* __restrict__ y, const double* __restrict__ V, const double* __restrict__ partial,
                               int blocks, int k, int64_t n, double* __restrict__ h)
{
    __shared__ double c[kMaxCombine];
    if (threadIdx.x < k) {
        double acc = 0.0;
#pragma unroll 4
        for (int b = 0; b < blocks; ++b) acc += partial[(int64_t)threadIdx.x * blocks + b];
        c[threadIdx.x] = -acc;
        if (blockIdx.x == 0) h[threadIdx.x] = acc;
    }
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    double s = 0.0;
#pragma unroll 4
    for (int j = 0; j < k; ++j) s = fma(c[j], V[(int64_t)j * n + i], s);
    y[i] += s;
}

// y[i] = x[i] / d[i]
__global__ void divide_kernel(double* __restrict__ y, const double* __restrict__ x, const double* __restrict__ d, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) y[i] = x[i] / d[i];
}

__global__ void reset_near_count_kernel(DevCounters* c) { c->near_count = 0ull; }

// everything the list pass and the near stage count; the far field's term counts stay
__global__ void reset_near_stage_kernel(DevCounters* c)
{
    c->near_count = 0ull;
    c->cursor = 0ull;
    c->leaves = 0ull;
    c->cap_hits = 0ull;
    c->on_surface = 0ull;
    c->max_depth = 0ull;
    c->visit_limit_hits = 0ull;
    c->heavy_cursor = 0ull;
}

hipError_t launch_reset_near_stage(DevCounters* c, hipStream_t s)
{
    reset_near_stage_kernel<<<1, 1, 0, s>>>(c);
    return hipGetLastError();
}

hipError_t launch_reset_near_count(DevCounters* c, hipStream_t s)
{
    reset_near_count_kernel<<<1, 1, 0, s>>>(c);
    return hipGetLastError();
}

hipError_t launch_zero_counters(DevCounters* c, hipStream_t s)
{
    zero_counters_kernel<<<1, 64, 0, s>>>(c);
    return hipGetLastError();
}

hipError_t launch_self_diag(const Elements& el, double K, double* diag, hipStream_t s)
{
    if (el.ne <= 0) return hipSuccess;
    self_diag_kernel<<<(unsigned)((el.ne + 255) / 256), 256, 0, s>>>(el, K, diag);
    return hipGetLastError();
}

hipError_t launch_multi_dot(const double* V, int k, int64_t n, const double* w, double* partial, int blocks, hipStream_t s)
{
    if (k < 1) return hipSuccess;
    multi_dot_kernel<<<dim3((unsigned)blocks, (unsigned)k), 256, 0, s>>>(V, n, w, partial);
    return hipGetLastError();
}

hipError_t launch_combine(double* y, double a, const double* V, const double* c, int k, int64_t n, const double* d,
                          hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (k < 0 || k > kMaxCombine) return hipErrorInvalidValue;
    CombineCoef coef;
    for (int j = 0; j < k; ++j) coef.c[j] = c[j];
    combine_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(y, a, V, coef, k, n, d);
    return hipGetLastError();
}

hipError_t launch_project(double* y, const double* V, const double* partial, int blocks, int k, int64_t n, double* h,
                          hipStream_t s)
{
    if (n <= 0 || k < 1) return hipSuccess;
    if (k > kMaxCombine) return hipErrorInvalidValue;
    project_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(y, V, partial, blocks, k, n, h);
    return hipGetLastError();
}

hipError_t launch_divide(double* y, const double* x, const double* d, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    divide_kernel<<<(unsigned)((n + 255) / 256), 256, 0, s>>>(y, x, d, n);
    return hipGetLastError();
}

}  // namespace bemc

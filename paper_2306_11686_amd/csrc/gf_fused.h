// gf_fused.h -- several sweeps of a stencil program per pass over the grid
// (temporal blocking) for the persistent kernel. Included only by
// gf_kernels.hip, after its wavefront shifts.
//
// A program whose body is one Jacobi region, scalar steps and the SWAP of the
// region's two grids is a chain of sweeps u^0, u^1, .., u^S in which sweep k
// reads buffer k mod 2 and writes the other. Only u^S and u^(S-1) are left in
// memory at the end, so a pass may read u^k, compute M sweeps in registers
// and write u^(k+M) alone: one read and one write of the grid, one grid
// barrier and one hand-over of the reduction per M sweeps instead of per
// sweep. M is odd, so u^(k+M) lands in the buffer the sequence would have
// put it in, and the last sweep is a pass of its own, so that u^(S-1) stays
// in the other buffer. Every point goes through the same operations in the
// same order as sweep by sweep (bit-exact), and every sweep's reduction is
// taken over the same points.
//
// Sweep by sweep the 2D stencil is bound by HBM on large grids and batches,
// and by the barrier, the reduction and the serial steps on small grids.
// Fused it moves a fifth of the bytes. Measured, sweep by sweep and fused: 256
// uneven instances, 50 sweeps, 28.4 and 6.7 ms; 256^2 with printf, 100 sweeps,
// 1,246 and 290 us. The instances' eight passes move 25.4 GB (20.7 without
// halos) at 3.8 TB/s with 39 % of the vector units' issue used (1.64e9
// instructions of four cycles), so neither bounds them: the latency of a
// march at three wavefronts per SIMD does, and the slowest group.
//
// Points of the outer layer are never written by a sweep, so u^s and u^(s-2)
// agree there, in whichever buffers they are: a stage takes the values of the
// outer layer from two stages earlier (the first stage from the destination
// buffer), also where the two buffers' outer layers differ.
#pragma once

namespace gf {

// 16-byte accesses of two columns; rows of an odd-sided grid start on 8-byte
// boundaries, which gfx950's dwordx4 accesses take.
typedef double gf_d2u __attribute__((ext_vector_type(2), aligned(8)));

// A row's address as an opaque scalar, so that accesses use it as their
// scalar base with the lane's fixed 32-bit offset (left alone, the compiler
// keeps a 64-bit address per lane for every access of the unrolled march).
template <typename V, typename T>
__device__ __forceinline__ GF_GLOBAL V *row_at(GF_GLOBAL T *p, uint32_t byte)
{
    // the offset too: its extension to 64 bits has to stay beside the access
    asm("" : "+s"(p), "+v"(byte));
    return (GF_GLOBAL V *)((GF_GLOBAL const char *)p + byte);
}

// Values of a pass's reductions over one work item or all of them.
template <int OP, int M>
__device__ __forceinline__ void wave_reduce_m(double (&v)[M])
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1)
#pragma unroll
        for (int s = 0; s < M; ++s)
            v[s] = RedOp<OP>::apply(v[s], __shfl_xor(v[s], off, kWave));
}

// M reductions at once over p[s * n + i], i < n, in a fixed order (strided
// per thread, then the wavefronts in order). lds: M doubles per wavefront.
// out[s] (LDS) holds the values when the workgroup returns.
template <int OP, int M>
__device__ __forceinline__ void reduce_partials_m(const double *p, int64_t n, double *lds, double *out)
{
    double acc[M];
#pragma unroll
    for (int s = 0; s < M; ++s)
        acc[s] = RedOp<OP>::identity();
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x)
#pragma unroll
        for (int s = 0; s < M; ++s)
            acc[s] = RedOp<OP>::apply(acc[s], p[s * n + i]);
    wave_reduce_m<OP, M>(acc);
    const int wid = threadIdx.x / kWave, nw = blockDim.x / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0)
#pragma unroll
        for (int s = 0; s < M; ++s)
            lds[wid * M + s] = acc[s];
    __syncthreads();
    if (threadIdx.x < M) {
        double v = lds[threadIdx.x];
        for (int w = 1; w < nw; ++w)
            v = RedOp<OP>::apply(v, lds[w * M + threadIdx.x]);
        out[threadIdx.x] = v;
    }
    __syncthreads();
}

// ---------------------------------------------------------------------------
// 2D. A work item belongs to one wavefront: 128 adjacent columns (two per
// lane), a segment of `rows` output rows. The wavefront marches down the
// rows; when row y arrives, stage s (s = 1 .. M) computes row y - s of sweep
// k + s from the rows y-s-1, y-s, y-s+1 of stage s-1, all in registers, with
// the x-neighbours taken from the adjacent lanes. Columns next to the
// wavefront's ends go wrong one per stage, so items overlap by M columns on
// each side, and by M rows above and below; wavefronts share nothing.
// ---------------------------------------------------------------------------

constexpr int kJ2fAhead = 3;              // rows in flight
constexpr int kJ2fRing = kJ2fAhead + 3;   // stage 0's rows; a multiple of 3, the other stages' period

struct J2fGeom {
    int32_t chunks;   // items across a row
    int32_t width;    // output columns per item (even)
    int32_t rows;     // output rows per item
    int64_t segs;     // items down the grid
    int64_t items;
};

// Items of 128 loaded columns across an n-column row when M columns are lost
// on an inner side, and the output columns of each.
__host__ __device__ inline void j2f_chunks(int64_t n, int M, int32_t *chunks, int32_t *width)
{
    const int64_t halo = (M + 1) & ~1;   // whole lanes lost on an inner side
    const int64_t cols = (n + 1) & ~(int64_t)1;
    int64_t c = 1;
    if (cols > 128) {
        c = 2;
        if (cols > 2 * (128 - halo))
            c = (cols + (128 - 2 * halo) - 1) / (128 - 2 * halo);
    }
    *chunks = (int32_t)c;
    *width = (int32_t)(((cols + c - 1) / c + 1) & ~(int64_t)1);
}

__host__ __device__ inline J2fGeom j2f_geom(int64_t n, int M)
{
    J2fGeom g;
    j2f_chunks(n, M, &g.chunks, &g.width);
    // long segments repeat less at their ends (M rows of the neighbours on
    // each side), short ones give a small grid more wavefronts
    const int64_t r = n / 32;
    g.rows = (int32_t)(r < 8 ? 8 : (r > 64 ? 64 : r));
    g.segs = (n - 2 + g.rows - 1) / g.rows;
    g.items = g.chunks * g.segs;
    return g;
}

// Output rows [y0, y1) of u^(k+M) from u = u^k; w holds the other buffer
// (outer layer of the odd stages, output). x0: the wavefront's first column
// (even), [xa, xb): its output columns (even bounds). acc[s] (s < M): the
// lane's sum of squared differences of sweep k + s + 1 over its output
// points. XE: the 128 columns include column 0 or n-1.
// Every load is issued unconditionally, rows past the last one read again:
// with loads under a branch the compiler cannot count what is in flight and
// waits for all of it at every row (the batch of 256 instances: a fifth
// slower).
template <int M, bool XE>
__device__ __forceinline__ void j2f_tile(GF_GLOBAL const double *__restrict__ u, GF_GLOBAL double *w, int32_t n,
                                         int32_t x0, int32_t xa, int32_t xb, int32_t y0, int32_t y1,
                                         double (&acc)[M])
{
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t x = x0 + 2 * lane;
    // lanes past the row's end load its last pair and are never used
    const uint32_t xs = 8u * (uint32_t)(XE && x > n - 2 ? n - 2 : x);
    const bool lone = XE && x == n - 1;               // odd n: column n-1 alone, second of its pair
    const bool bx = XE && (x == 0 || x == n - 1);     // first value is of the outer layer
    const bool by = XE && x + 1 == n - 1;             // second value is
    const bool zy = by || lone;                       // second value takes no part in the sum
    const bool mine = x >= xa && x < xb && x < n;
    const uint32_t xe = 8u * (uint32_t)(bx ? x : (by ? x + 1 : 0));  // the lane's outer column
    const int32_t ya = y0 - M > 0 ? y0 - M : 0;                      // first row read
    const int32_t yb = y1 - 1 + M < n - 1 ? y1 - 1 + M : n - 1;      // last row read
    const int32_t ye = y1 - 1 + M;                                   // last step
    const int64_t pitch = n;
    auto ld = [&](int32_t y) -> gf_d2 {
        const gf_d2 v = *row_at<const gf_d2u>(u + (y < yb ? y : yb) * pitch, xs);
        if constexpr (XE)
            return gf_d2{lone ? v.y : v.x, v.y};
        return v;
    };
    // the lane's outer column in the other buffer, row y
    auto ldb = [&](int32_t y) -> double { return *row_at<const double>(w + (y < yb ? y : yb) * pitch, xe); };
    auto ldrow = [&](int32_t y) -> gf_d2 {  // an outer row of the other buffer
        const gf_d2 v = *row_at<const gf_d2u>(w + y * pitch, xs);
        return gf_d2{lone ? v.y : v.x, v.y};
    };
    gf_d2 ring[kJ2fRing];        // stage 0: rows of u^k, row ya + j in slot j mod the ring
    double bc[XE ? kJ2fRing : 1];
    gf_d2 st[M > 1 ? M - 1 : 1][3];  // stage s = 1 .. M-1: its last three rows
    const gf_d2 zero2 = {0.0, 0.0};
#pragma unroll
    for (int s = 0; s < M - 1; ++s)
#pragma unroll
        for (int j = 0; j < 3; ++j)
            st[s][j] = zero2;
    // the outer row in the other buffer: the first row, later the last one
    // (used by segments that reach it)
    gf_d2 eb = ldrow(0);
#pragma unroll
    for (int j = 0; j < kJ2fRing; ++j) {
        ring[j] = j < kJ2fAhead ? ld(ya + j) : zero2;
        if constexpr (XE)
            bc[j] = j < kJ2fAhead ? ldb(ya + j) : 0.0;
    }
    // One step: row y arrives in slot k. The checks on the stages' rows are
    // scalar; a second version of the steps without them (for the middle of a
    // segment) doubled the code and, merged with this one in the loop, spilled.
    auto step = [&](auto kc, int32_t y) {
        constexpr int k = decltype(kc)::value;
        ring[(k + kJ2fAhead) % kJ2fRing] = ld(y + kJ2fAhead);
        if constexpr (XE)
            bc[(k + kJ2fAhead) % kJ2fRing] = ldb(y + kJ2fAhead);
#pragma unroll
        for (int s = 1; s <= M; ++s) {
            const int32_t r = y - s;
            // stage s-1's rows r-1, r, r+1
            const gf_d2 up = s == 1 ? ring[(k + kJ2fRing - 2) % kJ2fRing] : st[s >= 2 ? s - 2 : 0][(k + 1) % 3];
            const gf_d2 c = s == 1 ? ring[(k + kJ2fRing - 1) % kJ2fRing] : st[s >= 2 ? s - 2 : 0][(k + 2) % 3];
            const gf_d2 dn = s == 1 ? ring[k] : st[s >= 2 ? s - 2 : 0][k % 3];
            gf_d2 out;
            const int32_t lo = y0 - (M - s) > 0 ? y0 - (M - s) : 0;
            const int32_t hi = y1 - 1 + (M - s) < n - 1 ? y1 - 1 + (M - s) : n - 1;
            if (r < lo || r > hi)
                continue;
            gf_d2 prev = zero2;  // the same row two stages earlier
            if (s >= 3)
                prev = st[s >= 3 ? s - 3 : 0][(k + 1) % 3];
            else if (s == 2)
                prev = ring[(k + kJ2fRing - 2) % kJ2fRing];
            if (r == 0 || r == n - 1) {
                out = s == 1 ? eb : prev;
            } else {
                const double xl = wave_shr1(c.y);
                const double xr = wave_shl1(c.x);
                out.x = ((xl + c.y) + (up.x + dn.x)) * 0.25;
                out.y = ((c.x + xr) + (up.y + dn.y)) * 0.25;
                if constexpr (XE) {
                    const double b = s == 1 ? bc[(k + kJ2fRing - 1) % kJ2fRing] : 0.0;
                    out.x = bx ? (s == 1 ? b : prev.x) : out.x;
                    out.y = by ? (s == 1 ? b : prev.y) : out.y;
                }
                if (r >= y0 && r < y1) {
                    double dx = out.x - c.x, dy = out.y - c.y;
                    if constexpr (XE) {
                        dx = bx ? 0.0 : dx;
                        dy = zy ? 0.0 : dy;
                    }
                    acc[s - 1] = __builtin_fma(dx, dx, acc[s - 1]);
                    acc[s - 1] = __builtin_fma(dy, dy, acc[s - 1]);
                    // accumulate here: sunk to the end of the unrolled steps,
                    // the sums keep every step's rows in registers
                    asm volatile("" : "+v"(acc[s - 1]));
                    if (s == M && mine) {
                        GF_GLOBAL double *o = row_at<double>(w + r * pitch, xs);
                        if (!XE || (!bx && !by))
                            __builtin_nontemporal_store(out, (GF_GLOBAL gf_d2u *)o);
                        else if (!bx)
                            __builtin_nontemporal_store(out.x, o);
                        else if (!zy)
                            __builtin_nontemporal_store(out.y, o + 1);
                    }
                }
            }
            if (s < M)
                st[s < M ? s - 1 : 0][k % 3] = out;
        }
    };
    for (int32_t y = ya;;) {
        // past the first row at every stage: from here the outer row is the
        // last one (the first stage reaches it at step n)
        if (y > M)
            eb = ldrow(n - 1);
        step(std::integral_constant<int, 0>{}, y);
        if (++y > ye)
            break;
        step(std::integral_constant<int, 1>{}, y);
        if (++y > ye)
            break;
        step(std::integral_constant<int, 2>{}, y);
        if (++y > ye)
            break;
        step(std::integral_constant<int, 3>{}, y);
        if (++y > ye)
            break;
        step(std::integral_constant<int, 4>{}, y);
        if (++y > ye)
            break;
        step(std::integral_constant<int, 5>{}, y);
        if (++y > ye)
            break;
    }
    static_assert(kJ2fRing == 6, "steps written out above");
#pragma unroll
    for (int s = 0; s < M; ++s)
        acc[s] = mine ? acc[s] : 0.0;
}

template <int M>
__device__ __forceinline__ void j2f_item(const double *u_, double *w_, int64_t n, int64_t item,
                                         double (&acc)[M])
{
    const J2fGeom g = j2f_geom(n, M);
    const int64_t c = item % g.chunks;
    const int64_t y0 = 1 + (item / g.chunks) * g.rows;
    const int64_t y1 = y0 + g.rows < n - 1 ? y0 + g.rows : n - 1;
    const int64_t halo = (M + 1) & ~1;
    const int64_t cols = (n + 1) & ~(int64_t)1;
    const int64_t xa = c * g.width;
    const int64_t xb = xa + g.width;
    const int64_t xmax = cols > 128 ? cols - 128 : 0;
    int64_t x0 = xa - halo > 0 ? xa - halo : 0;
    x0 = x0 < xmax ? x0 : xmax;
#pragma unroll
    for (int s = 0; s < M; ++s)
        acc[s] = 0.0;
    if (x0 == 0 || x0 + 128 >= n)
        j2f_tile<M, true>(gptr(u_), gptr(w_), (int32_t)n, (int32_t)x0, (int32_t)xa, (int32_t)xb, (int32_t)y0,
                          (int32_t)y1, acc);
    else
        j2f_tile<M, false>(gptr(u_), gptr(w_), (int32_t)n, (int32_t)x0, (int32_t)xa, (int32_t)xb, (int32_t)y0,
                           (int32_t)y1, acc);
}

// ---------------------------------------------------------------------------
// 3D. A workgroup owns 128 columns (two per lane) by 32 rows, four per
// wavefront, and marches z. When plane z arrives, stage s computes plane
// z - s of sweep k + s from stage s-1's planes z-s-1, z-s, z-s+1, all in
// registers. The rows above and below a wavefront's own are the neighbouring
// wavefronts': each lays the edge rows of every stage's newest plane in LDS
// at the end of a step, and they are read a step later, when that plane is
// the middle one, so that one barrier per step is enough. The tile's outermost
// rows go wrong one per stage, like the columns: it writes 32 - 2 M rows. A
// plane's rows are requested as soon as the registers of the plane three
// before are free, one step ahead of their use.
// 512^3, 100 sweeps: 44.9 ms a sweep at a time; 20.6 with every wavefront
// computing the rows around its three output rows itself (5 rows of work for
// one output row and three sweeps); 16.3 to 16.7 so (3.7). About 490 us a
// pass of three sweeps, 2.5 GB (reads 1.41, writes 1.08; an eighth of it
// halos) at 5 TB/s, with 47 % of the vector units' issue used: bound by HBM and
// by the steps' latency at two wavefronts per SIMD.
// Where the two buffers' outer layers agree (the kernel compares them first) a
// point of the outer layer keeps its value at every stage. Where they differ
// (DIFF), sweep k + s leaves there what its buffer holds: the lanes that hold
// an outer column request its values at the start of a step, outer rows and
// planes are read as they come. 30 sweeps, us, agreeing, differing, a sweep at
// a time with the fixed tile: side 64 238 / 260 / 4,938, 256 1,042 / 1,383 /
// 5,655, 512 5,865 / 8,390 / 13,440. One sweep per pass, as differing layers
// took at first: 313 / 2,197 / 12,700. All outer values read where they are
// needed: 13,200 at 512, and 8 % slower where they agree.
// ---------------------------------------------------------------------------

constexpr int kJ3fRows = 4;    // rows per wavefront
constexpr int kJ3fWaves = 8;   // wavefronts of a workgroup, along y
constexpr int kJ3fTile = kJ3fRows * kJ3fWaves;

struct J3fGeom {
    int32_t chunks, width;  // items across a row, output columns of one (even)
    int32_t yt, height;     // workgroup tiles along y, output rows of one
    int32_t zlen, zs;       // planes per segment, segments
    int64_t items;          // workgroup items
};

__host__ __device__ inline J3fGeom j3f_geom(int64_t n, int M, int32_t zlen)
{
    J3fGeom g;
    j2f_chunks(n, M, &g.chunks, &g.width);
    const int32_t in = n > 2 ? (int32_t)(n - 2) : 0, most = kJ3fTile - 2 * M;
    const int32_t tiles = in > 0 ? (in + most - 1) / most : 1;
    g.height = in > 0 ? (in + tiles - 1) / tiles : 1;
    g.yt = (in + g.height - 1) / g.height;
    g.zlen = zlen;
    g.zs = (int32_t)((in + zlen - 1) / zlen);
    g.items = (int64_t)g.chunks * g.yt * g.zs;
    return g;
}

// Planes per segment for a pass of M sweeps shared by G workgroups: the
// fewest plane steps of the slowest workgroup (a segment repeats M planes on
// each side), and one more step per 64 workgroups for the barrier.
__host__ __device__ inline int32_t j3f_zlen(int64_t n, int M, int64_t G)
{
    const int64_t in = n > 2 ? n - 2 : 1;
    int64_t best = 0, best_cost = 0;
    for (int64_t zs = 1; zs <= in && zs <= kFusedMaxSegs3; ++zs) {
        const int64_t zl = (in + zs - 1) / zs;
        const int64_t items = j3f_geom(n, M, (int32_t)zl).items;
        const int64_t rounds = (items + G - 1) / G;
        const int64_t cost = rounds * (zl + 2 * M) * 64 + (items < G ? items : G);
        if (best == 0 || cost < best_cost) {
            best = zl;
            best_cost = cost;
        }
    }
    return (int32_t)best;
}

// Whether the outer layers of the two n-sided 3D grids hold the same bits,
// in the points of worker `worker` of G.
__device__ __forceinline__ bool outer3_agrees(GF_GLOBAL const double *a_, GF_GLOBAL const double *b_, int64_t n,
                                              int64_t worker, int64_t G)
{
    GF_GLOBAL const uint64_t *a = (GF_GLOBAL const uint64_t *)a_;
    GF_GLOBAL const uint64_t *b = (GF_GLOBAL const uint64_t *)b_;
    const int64_t sq = n * n, far = n - 1;
    uint64_t diff = 0;
    for (int64_t i = worker * blockDim.x + threadIdx.x; i < sq; i += G * blockDim.x) {
        const int64_t p = i / n, q = i - p * n;
        diff |= (a[i] ^ b[i]) | (a[far * sq + i] ^ b[far * sq + i]);                          // z faces
        diff |= (a[p * sq + q] ^ b[p * sq + q]) | (a[p * sq + far * n + q] ^ b[p * sq + far * n + q]);  // y faces
        diff |= (a[i * n] ^ b[i * n]) | (a[i * n + far] ^ b[i * n + far]);                    // x faces
    }
    return diff == 0;
}

// Edge rows of the planes that the stages of a workgroup's wavefronts read
// next: [parity of the step][stage][wavefront][first, last row][lane].
template <int M>
struct J3fEdges {
    gf_d2 row[2][M][kJ3fWaves][2][kWave];
};

// Planes [z0, z1), rows [ylo, yhi) of u^(k+M), by a wavefront that holds rows
// [r0, r0 + kJ3fRows). EDGE: the tile's rows or columns touch the outer
// layer. DIFF: the two buffers' outer layers differ. acc[s]: the lane's
// max |difference| of sweep k + s + 1.
template <int M, bool EDGE, bool DIFF>
__device__ __forceinline__ void j3f_tile(GF_GLOBAL const double *__restrict__ u, GF_GLOBAL double *__restrict__ w,
                                         J3fEdges<M> &edges, int32_t n, int32_t x0, int32_t xa, int32_t xb, int32_t r0,
                                         int32_t ylo, int32_t yhi, int32_t z0, int32_t z1, int wv, double (&acc)[M])
{
    constexpr int TY = kJ3fRows;
    const int lane = threadIdx.x & (kWave - 1);
    const int32_t x = x0 + 2 * lane;
    const uint32_t xs = 8u * (uint32_t)(EDGE && x > n - 2 ? n - 2 : x);
    const bool lone = EDGE && x == n - 1;
    const bool bx = EDGE && (x == 0 || x == n - 1);
    const bool by = EDGE && x + 1 == n - 1;
    const bool zy = by || lone;
    const bool mine = x >= xa && x < xb && x < n;
    const int64_t pitch = n, plane = (int64_t)n * n;
    const int32_t za = z0 - M > 0 ? z0 - M : 0;                    // first plane read
    const int32_t zb = z1 - 1 + M < n - 1 ? z1 - 1 + M : n - 1;    // last plane read
    const int32_t ze = z1 - 1 + M;                                 // last step
    // the wavefronts above and below (at the tile's ends: any row, never used)
    const int wu = wv > 0 ? wv - 1 : 0, wd = wv + 1 < kJ3fWaves ? wv + 1 : wv;
    auto ld = [&](int32_t z, int j) -> gf_d2 {
        int32_t y = r0 + j;
        if constexpr (EDGE)
            y = y > n - 1 ? n - 1 : y;
        const gf_d2 v = *row_at<const gf_d2u>(u + (z < zb ? z : zb) * plane + y * pitch, xs);
        if constexpr (EDGE)
            return gf_d2{lone ? v.y : v.x, v.y};
        return v;
    };
    // DIFF: row y of plane z of sweep k + s, at points of the outer layer
    auto clamped = [&](int32_t v) -> int32_t { return v < 0 ? 0 : (v > n - 1 ? n - 1 : v); };
    auto ld_outer = [&](int s, int32_t z, int32_t y) -> gf_d2 {
        const gf_d2 v = *row_at<const gf_d2u>((s & 1 ? w : u) + clamped(z) * plane + clamped(y) * pitch, xs);
        return gf_d2{lone ? v.y : v.x, v.y};
    };
    const uint32_t xe = 8u * (uint32_t)(by ? x + 1 : (EDGE && x > n - 1 ? n - 1 : x));  // the lane's outer column
    const gf_d2 zero2 = {0.0, 0.0};
    // q[s][slot][row]: stage s's planes
    gf_d2 q[M][3][TY];
#pragma unroll
    for (int s = 0; s < M; ++s)
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
            for (int j = 0; j < TY; ++j)
                q[s][k][j] = zero2;
#pragma unroll
    for (int j = 0; j < TY; ++j)
        q[0][0][j] = ld(za, j);
    const double c6 = 1.0 / 6.0;
    // one step: plane z is in slot k of stage 0. ENDS: a stage may be at the
    // first or the last plane
    auto step = [&](auto kc, auto ends, int32_t plane_in) {
        const int32_t z = __builtin_amdgcn_readfirstlane(plane_in);
        constexpr int k = decltype(kc)::value;
        constexpr bool ENDS = decltype(ends)::value;
        constexpr int kc1 = (k + 2) % 3, km = (k + 1) % 3;  // the planes one and two before
        double xo[M > 1 ? M - 1 : 1][TY];  // stage s + 1's values in the lane's outer column
        if constexpr (DIFF && EDGE)
#pragma unroll
            for (int s = 1; s < M; ++s)
#pragma unroll
                for (int j = 0; j < TY; ++j)
                    xo[s - 1][j] = *row_at<const double>((s & 1 ? w : u) + clamped(z - s) * plane +
                                                             clamped(r0 + j) * pitch, xe);
        __syncthreads();  // the edge rows of the step before are in LDS, those of the one before that free
        gf_d2 nu[M], nd[M];
#pragma unroll
        for (int s = 0; s < M; ++s) {
            nu[s] = edges.row[(z + 1) & 1][s][wu][1][lane];
            nd[s] = edges.row[(z + 1) & 1][s][wd][0][lane];
        }
        gf_d2 fin[TY];
#pragma unroll
        for (int s = 1; s <= M; ++s)
#pragma unroll
            for (int i = 0; i < TY; ++i) {
                // the rows that need the neighbours' last
                const int j = i < TY - 2 ? i + 1 : (i == TY - 2 ? 0 : TY - 1);
                const gf_d2 c = q[s - 1][kc1][j];
                const gf_d2 up = j > 0 ? q[s - 1][kc1][j > 0 ? j - 1 : 0] : nu[s - 1];
                const gf_d2 dn = j + 1 < TY ? q[s - 1][kc1][j + 1 < TY ? j + 1 : 0] : nd[s - 1];
                const gf_d2 zm = q[s - 1][km][j], zp = q[s - 1][k][j];
                const double xl = wave_shr1(c.y);
                const double xr = wave_shl1(c.x);
                gf_d2 out;
                out.x = (((xl + c.y) + (up.x + dn.x)) + (zm.x + zp.x)) * c6;
                out.y = (((c.x + xr) + (up.y + dn.y)) + (zm.y + zp.y)) * c6;
                if constexpr (EDGE || ENDS) {
                    const int32_t y = r0 + j;
                    const bool flat = y <= 0 || y >= n - 1 || z - s <= 0 || z - s >= n - 1;
                    if constexpr (DIFF) {
                        if (s < M) {
                            if constexpr (EDGE) {
                                out.x = bx ? xo[s < M ? s - 1 : 0][j] : out.x;
                                out.y = by ? xo[s < M ? s - 1 : 0][j] : out.y;
                            }
                            if (flat)
                                out = ld_outer(s, z - s, y);
                        }
                    } else {
                        out.x = (bx || flat) ? c.x : out.x;
                        out.y = (by || flat) ? c.y : out.y;
                    }
                }
                // computed here: sunk towards its use in the next steps, the
                // value keeps all of its inputs in registers
                asm volatile("" : "+v"(out.x), "+v"(out.y));
                if (s < M)
                    q[s < M ? s : 0][k][j] = out;
                else
                    fin[j] = out;
                // stage 0's plane z-2 is done with
                if (s == 1)
                    q[0][km][j] = ld(z + 1, j);
            }
#pragma unroll
        for (int s = 0; s < M; ++s) {
            edges.row[z & 1][s][wv][0][lane] = q[s][k][0];
            edges.row[z & 1][s][wv][1][lane] = q[s][k][TY - 1];
        }
        // the output rows' differences, planes of this segment
#pragma unroll
        for (int s = 1; s <= M; ++s)
            if (z - s >= z0 && z - s < z1) {
#pragma unroll
                for (int j = 0; j < TY; ++j) {
                    if (r0 + j < ylo || r0 + j >= yhi)
                        continue;
                    const gf_d2 o = s < M ? q[s < M ? s : 0][k][j] : fin[j];
                    const gf_d2 c = q[s - 1][kc1][j];
                    double dx = __builtin_fabs(o.x - c.x), dy = __builtin_fabs(o.y - c.y);
                    if constexpr (EDGE) {
                        dx = bx ? -INFINITY : dx;
                        dy = zy ? -INFINITY : dy;
                    }
                    acc[s - 1] = __builtin_fmax(acc[s - 1], __builtin_fmax(dx, dy));
                    if (s == M && mine) {
                        GF_GLOBAL double *p = row_at<double>(w + (z - M) * plane + (r0 + j) * pitch, xs);
                        if (!EDGE || (!bx && !by))
                            __builtin_nontemporal_store(o, (GF_GLOBAL gf_d2u *)p);
                        else if (!bx)
                            __builtin_nontemporal_store(o.x, p);
                        else if (!zy)
                            __builtin_nontemporal_store(o.y, p + 1);
                    }
                }
            }
    };
    auto any_step = [&](auto kc, int32_t z) {
        if (EDGE || z <= M || z >= n)
            step(kc, std::true_type{}, z);
        else
            step(kc, std::false_type{}, z);
    };
    for (int32_t z = za;;) {
        any_step(std::integral_constant<int, 0>{}, z);
        if (++z > ze)
            break;
        any_step(std::integral_constant<int, 1>{}, z);
        if (++z > ze)
            break;
        any_step(std::integral_constant<int, 2>{}, z);
        if (++z > ze)
            break;
    }
#pragma unroll
    for (int s = 0; s < M; ++s)
        acc[s] = mine ? acc[s] : -INFINITY;
}

// One workgroup item: wavefront wv's rows.
template <int M, bool DIFF>
__device__ __forceinline__ void j3f_item(const double *u_, double *w_, J3fEdges<M> &edges, int64_t n, int32_t zlen,
                                         int64_t item, int wv, double (&acc)[M])
{
    const J3fGeom g = j3f_geom(n, M, zlen);
    const int64_t c = item % g.chunks;
    const int64_t rest = item / g.chunks;
    const int64_t yt = rest % g.yt;
    const int64_t zi = rest / g.yt;
    const int64_t z0 = 1 + zi * g.zlen;
    const int64_t z1 = z0 + g.zlen < n - 1 ? z0 + g.zlen : n - 1;
    const int64_t ylo = 1 + yt * g.height;
    const int64_t yhi = ylo + g.height < n - 1 ? ylo + g.height : n - 1;
    const int64_t ymax = n > kJ3fTile ? n - kJ3fTile : 0;
    int64_t rt = ylo - M > 0 ? ylo - M : 0;  // the tile's first row
    rt = rt < ymax ? rt : ymax;
    const int64_t halo = (M + 1) & ~1;
    const int64_t cols = (n + 1) & ~(int64_t)1;
    const int64_t xa = c * g.width;
    const int64_t xmax = cols > 128 ? cols - 128 : 0;
    int64_t x0 = xa - halo > 0 ? xa - halo : 0;
    x0 = x0 < xmax ? x0 : xmax;
#pragma unroll
    for (int s = 0; s < M; ++s)
        acc[s] = -INFINITY;
    // the rows the stages compute, and the columns they load; the same for all
    // wavefronts of the workgroup, which have to meet at one barrier (not at
    // the two versions' own)
    const bool edge = x0 == 0 || x0 + 128 >= n || rt == 0 || rt + kJ3fTile >= n;
    // uniform: kept in scalar registers
    auto uni = [](int64_t v) -> int32_t { return __builtin_amdgcn_readfirstlane((int32_t)v); };
    const int32_t side = uni(n), xs = uni(x0), xl = uni(xa), xh = uni(xa + g.width),
                  rs = uni(rt) + wv * kJ3fRows, yl = uni(ylo), yh = uni(yhi), zl = uni(z0), zh = uni(z1);
    if (__builtin_amdgcn_readfirstlane(edge))
        j3f_tile<M, true, DIFF>(gptr(u_), gptr(w_), edges, side, xs, xl, xh, rs, yl, yh, zl, zh, wv, acc);
    else
        j3f_tile<M, false, DIFF>(gptr(u_), gptr(w_), edges, side, xs, xl, xh, rs, yl, yh, zl, zh, wv, acc);
}

}  // namespace gf

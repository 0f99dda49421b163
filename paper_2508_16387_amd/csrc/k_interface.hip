// k_interface.hip -- interface-face work queue, FIVER fluxes and the phase
// update.
//
// FIVER (section "Spatial discretization of governing equations", eq.
// 1DRiemannProblem): at a face whose two cells hold different materials the
// flux is not one HLLC flux but two one-sided fluxes built on the exact
// solution of the two-material Riemann problem along the face normal.  Those
// faces are a thin sheet (well under 1% of all faces), so they are gathered
// into a dense queue once per step (material ids are frozen during a step)
// and solved by one thread each, away from the bulk stage kernel whose
// wavefronts would otherwise diverge on the Newton iteration.
//
// Queue order is ascending face id f = 3c + d (face between cell c and its
// +d neighbour); the compaction is deterministic (counts per chunk of cells,
// then each block adds up the counts before its own and writes its faces with
// wavefront prefix sums), so the queue is bit-identical from run to run.
//
// Launches of a single-grid step besides its bulk stages: k_step_begin (the
// phase update of the step before, the counts), then per Runge-Kutta stage
// one FIVER launch, the first of which also writes a rebuilt queue and opens
// the step.  Each is a chain of a few dependent memory accesses whatever its
// size, so a launch saved is its whole time saved: count, scan and scatter as
// launches of their own took 4.5 + 4.6 + 4.8 us of a 128^3 step that keeps its
// queue, where the two now take 4.3 and 1 more in the first FIVER launch, and
// 20.8 + 4.7 + 8.4 us, with 11.4 for that FIVER launch, where it is rebuilt:
// 17.1 + 19.2 now.  General EOS, 128^3 charge, whose queue is rebuilt in every
// step by a launch of its own: 25 + 5 + 10 -> 21 + 10 us.  The face -> slot
// map is written only at the faces of the new queue and read only at faces
// whose cells differ in material under the same frozen ids, so entries left
// from earlier queues are never read and need no clearing.
#include "m2c_device.h"
#include "m2c_internal.h"
#include "m2c_kernels.h"
#include "m2c_mlp_eos.h"
#include "m2c_mlp_infer.h"

namespace m2c {

// Interface-face bits of cell c: bit d set when the face towards the +d
// neighbour separates two materials.  A face on a non-periodic domain
// boundary is never an interface (the boundary image carries the boundary
// cell's material); a periodic axis wraps.  Cell indices fit in 32 bits
// (grids are limited to 2^29 cells).
// A lane walks its cells c, c + 64, c + 128, ... with their coordinates
// (i, j, k) advanced incrementally (no division per cell).
struct CellWalk {
    uint32_t c, i, j, k;
};

__device__ __forceinline__ void walk_start(const Grid& G, uint32_t c, CellWalk& w)
{
    const uint32_t nx = G.nx, sxy = nx * (uint32_t)G.ny;
    w.c = c;
    w.k = c / sxy;
    const uint32_t r = c - w.k * sxy;
    w.j = r / nx;
    w.i = r - w.j * nx;
}

__device__ __forceinline__ void walk_advance(const Grid& G, CellWalk& w, uint32_t step = 64u)
{
    const uint32_t nx = G.nx, ny = G.ny;
    w.c += step;
    w.i += step;
    while (w.i >= nx) {
        w.i -= nx;
        if (++w.j == ny) {
            w.j = 0;
            ++w.k;
        }
    }
}

__device__ __forceinline__ unsigned cell_face_bits(const Grid& G, const uint8_t* __restrict__ chi, const CellWalk& w)
{
    const uint32_t nx = G.nx, ny = G.ny, nz = G.nz, sxy = nx * ny;
    const uint32_t c = w.c, i = w.i, j = w.j, k = w.k;
    const uint8_t x = chi[c];
    unsigned bits = 0;
    if (G.act[0] && (i + 1 < nx || G.bc[1] == BC_PERIODIC)) {
        const uint32_t n = i + 1 < nx ? c + 1 : c - (nx - 1);
        if (chi[n] != x) bits |= 1u;
    }
    if (G.act[1] && (j + 1 < ny || G.bc[3] == BC_PERIODIC)) {
        const uint32_t n = j + 1 < ny ? c + nx : c - (ny - 1) * nx;
        if (chi[n] != x) bits |= 2u;
    }
    if (G.act[2] && (k + 1 < nz || G.bc[5] == BC_PERIODIC)) {
        const uint32_t n = k + 1 < nz ? c + sxy : c - (nz - 1) * sxy;
        if (chi[n] != x) bits |= 4u;
    }
    return bits;
}

// Cells of a compaction block: wave w owns the 64 * COMPACT_CELLS_PER_THREAD
// consecutive cells from blk * COMPACT_CELLS_PER_BLOCK + w * 64 *
// COMPACT_CELLS_PER_THREAD (how its lanes share them: lane_bits_* below), so
// the queue order over waves and blocks is ascending cell order.
__device__ __forceinline__ uint32_t compact_wave_base(int blk)
{
    return (uint32_t)blk * COMPACT_CELLS_PER_BLOCK + (threadIdx.x >> 6) * (64 * COMPACT_CELLS_PER_THREAD);
}

__device__ __forceinline__ int block_sum(int v, int* sRed)
{
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) sRed[w] = v;
    __syncthreads();
    int t = 0;
    for (int k = 0; k < (int)(blockDim.x >> 6); ++k) t += sRed[k];
    return t;
}

// Face bits of the lane's cells.  Byte path (any grid): in round e the lane
// takes cell wbase + 64 e + l, packed at bits 3e..3e+2.  Word path (nx a
// multiple of 4, ids 4-byte aligned): in round e the lane takes the four
// cells wbase + 256 e + 4 l + b (b = 0..3) with one aligned 32-bit load of
// their ids and one per neighbouring row, plane and (for b = 3) the next
// word, packed at bits 3(4e + b)...; a quarter of the memory instructions.
__device__ __forceinline__ bool compact_words(const Grid& G, const uint8_t* chi)
{
    return G.nx % 4 == 0 && ((uintptr_t)chi & 3u) == 0;
}

__device__ __forceinline__ uint64_t lane_bits_bytes(const Grid& G, const uint8_t* __restrict__ chi, uint32_t wbase,
                                                    int& cnt)
{
    const uint32_t N = (uint32_t)G.N;
    uint64_t packed = 0;
    cnt = 0;
    CellWalk cw;
    walk_start(G, wbase + (threadIdx.x & 63), cw);
#pragma unroll
    for (int e = 0; e < COMPACT_CELLS_PER_THREAD; ++e) {
        const unsigned bits = cw.c < N ? cell_face_bits(G, chi, cw) : 0u;
        walk_advance(G, cw);
        packed |= (uint64_t)bits << (3 * e);
        cnt += __popc(bits);
    }
    return packed;
}

__device__ __forceinline__ uint32_t ld_word(const uint8_t* __restrict__ chi, uint32_t c)
{
    return *reinterpret_cast<const uint32_t*>(chi + c);
}

__device__ __forceinline__ uint64_t lane_bits_words(const Grid& G, const uint8_t* __restrict__ chi, uint32_t wbase,
                                                    int& cnt)
{
    const uint32_t N = (uint32_t)G.N, nx = G.nx, ny = G.ny, nz = G.nz, sxy = nx * ny;
    const bool py = G.bc[3] == BC_PERIODIC, pz = G.bc[5] == BC_PERIODIC, px = G.bc[1] == BC_PERIODIC;
    uint64_t packed = 0;
    cnt = 0;
    CellWalk cw;
    walk_start(G, wbase + 4u * (threadIdx.x & 63), cw);
#pragma unroll
    for (int e = 0; e < COMPACT_CELLS_PER_THREAD / 4; ++e) {
        if (cw.c < N) {
            const uint32_t c = cw.c;
            const uint32_t d0 = ld_word(chi, c);
            // neighbour words (all 4-byte aligned since nx % 4 == 0)
            const bool hx = cw.i + 4 < nx || px;
            const bool hy = G.act[1] && (cw.j + 1 < ny || py);
            const bool hz = G.act[2] && (cw.k + 1 < nz || pz);
            const uint32_t dx = hx ? ld_word(chi, cw.i + 4 < nx ? c + 4 : c + 4 - nx) : 0u;
            const uint32_t dy = hy ? ld_word(chi, cw.j + 1 < ny ? c + nx : c - (ny - 1) * nx) : 0u;
            const uint32_t dz = hz ? ld_word(chi, cw.k + 1 < nz ? c + sxy : c - (nz - 1) * sxy) : 0u;
            const uint32_t nxw = (d0 >> 8) | (dx << 24);     // +x neighbour of each byte
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const uint32_t x = (d0 >> (8 * b)) & 0xffu;
                unsigned bits = 0;
                if ((b < 3 || hx) && ((nxw >> (8 * b)) & 0xffu) != x) bits |= 1u;
                if (hy && ((dy >> (8 * b)) & 0xffu) != x) bits |= 2u;
                if (hz && ((dz >> (8 * b)) & 0xffu) != x) bits |= 4u;
                packed |= (uint64_t)bits << (3 * (4 * e + b));
                cnt += __popc(bits);
            }
        }
        walk_advance(G, cw, 256u);
    }
    return packed;
}

// Compaction blocks [first, end) of a chunk.
__device__ __forceinline__ int2 chunk_blocks(const IfaceArgs& a, int chunk)
{
    const int per = compact_per_chunk(a.nblk);
    return make_int2(chunk * per, min(a.nblk, (chunk + 1) * per));
}

__device__ __forceinline__ void count_body(const IfaceArgs& a, int chunk)
{
    __shared__ int sRed[COMPACT_THREADS / 64];
    const int2 r = chunk_blocks(a, chunk);
    const bool words = compact_words(a.g, a.chi);
    int cnt = 0;
    for (int blk = r.x; blk < r.y; ++blk) {
        int k;
        if (words) (void)lane_bits_words(a.g, a.chi, compact_wave_base(blk), k);
        else (void)lane_bits_bytes(a.g, a.chi, compact_wave_base(blk), k);
        cnt += k;
    }
    const int t = block_sum(cnt, sRed);
    if (threadIdx.x == 0) a.blockcnt[chunk] = t;
}

// A step whose predecessor flipped no cell has the material ids the queue
// was built from (the last stage writes every id, and a flip is exactly a
// changed id), so the compaction keeps the queue and the face slots.  The
// decision is taken before the flip count is cleared, and recorded for the
// scatter.
__device__ __forceinline__ bool queue_kept(const DevScalars* sc) { return sc->qvalid && sc->nflip == 0; }

// Faces of the chunks [0, n), for every thread of the block.
__device__ __forceinline__ int count_prefix(const IfaceArgs& a, int n)
{
    __shared__ int sRed[COMPACT_THREADS / 64];
    int v = 0;
    for (int b = threadIdx.x; b < n; b += COMPACT_THREADS) v += a.blockcnt[b];
    __syncthreads();                              // sRed of an earlier call
    return block_sum(v, sRed);
}

// Length of a rebuilt queue.
__device__ __forceinline__ int count_total(const IfaceArgs& a) { return count_prefix(a, compact_chunks(a.nblk)); }

// Whether a step before the one being opened failed: an error that is not
// from the launch that opens it.
__device__ __forceinline__ bool failed_before(int err) { return err != 0 && err != ST_RIEMANN_OPENING; }

// An opening launch's error becomes an ordinary one, when that launch is over.
__device__ __forceinline__ void settle_error(DevScalars* sc, int err)
{
    if (err == ST_RIEMANN_OPENING) sc->err = ST_RIEMANN;
}

// End of a step (single grid) that no kernel reported an error of: counters
// and simulated time.
__device__ __forceinline__ void end_step_body(DevScalars* sc, int stages)
{
    sc->steps_done += 1;
    sc->t += sc->dt;
    sc->dt_last = sc->dt;
    sc->solves += (long long)sc->qlen * stages;
    sc->flips += sc->nflip;
}

// Start of a step (single grid): dt from the CFL rule (section "Time
// integration"; the rule itself is not printed, the reading is dt = CFL /
// max_i sum over the axes with more than one cell of (|V_d| + c)/h_d) or
// imposed; clear the accumulators that the step fills for the next step.
__device__ __forceinline__ void begin_step_body(DevScalars* sc, double cfl, double dt_fixed, double dt_imposed)
{
    double dt;
    if (dt_imposed > 0.0) dt = dt_imposed;
    else if (dt_fixed > 0.0) dt = dt_fixed;
    else dt = cfl / __longlong_as_double((long long)sc->lam_bits);
    sc->dt = dt;
    sc->lam_bits = 0ull;
    sc->nflip = 0;
}

// Opens a step in one block of the launch that follows k_step_begin: ends
// the previous step of the same m2c_step call (end_prev), forms dt (begin)
// and, when the queue was rebuilt, records its length.  The other blocks of
// the launch read none of what it writes.  It reads one word that they write:
// the error status, when the launch also solves the new step's faces and one
// of them fails.  Such a failure must not pass for one of the step being
// closed, whichever comes first, so the launch reports it as
// ST_RIEMANN_OPENING, which counts here as no failure.  An error left by
// earlier launches is never that code: k_step_begin, the launch before, and
// k_end_step, the last of a call, settle it.  All others only ask whether the
// status is 0.
// total: the length of a rebuilt queue (qreuse 0).
__device__ __forceinline__ void open_step(const IfaceArgs& a, const StepOpen& o, int total)
{
    if (threadIdx.x != 0) return;
    DevScalars* sc = a.sc;
    const bool rebuilt = !sc->qreuse;
    const bool failed = failed_before(sc->err);
    if (o.end_prev && !failed) end_step_body(sc, a.g.rk_stages);
    if (o.begin && !failed) begin_step_body(sc, a.g.cfl, a.g.dt_fixed, o.dt_imposed);
    if (!rebuilt) return;
    // (a queue past its capacity is not written, see scatter_body, nor solved)
    if (total > a.qcap) atomicCAS(&sc->err, 0, ST_OVERFLOW);
    sc->qlen = total > a.qcap ? 0 : total;
    sc->qvalid = failed || total > a.qcap ? 0 : 1;
}

__global__ void k_end_step(DevScalars* sc, int stages)
{
    const int err = sc->err;
    if (err == 0) end_step_body(sc, stages);
    settle_error(sc, err);
}

hipError_t launch_end_step(DevScalars* sc, int stages, hipStream_t s)
{
    hipLaunchKernelGGL(k_end_step, dim3(1), dim3(1), 0, s, sc, stages);
    return hipGetLastError();
}

// Writes the queue entries and face slots of compaction block blk, whose
// faces take the queue positions from base on (none where they would pass the
// queue's capacity); with PART only those at positions [from, to).  Returns
// the number of its faces.
template <bool PART = false>
__device__ __forceinline__ int scatter_body(const IfaceArgs& a, int blk, int base, int from = 0, int to = 0)
{
    __shared__ int sW[COMPACT_THREADS / 64];
    const uint32_t wbase = compact_wave_base(blk);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const bool words = compact_words(a.g, a.chi);
    int cnt = 0;
    const uint64_t packed = words ? lane_bits_words(a.g, a.chi, wbase, cnt) : lane_bits_bytes(a.g, a.chi, wbase, cnt);
    for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o);
    if (lane == 0) sW[w] = cnt;
    __syncthreads();
    int total = 0;
    for (int k = 0; k < COMPACT_THREADS / 64; ++k) total += sW[k];
    if ((long long)base + total > a.qcap) return total;
    if (cnt == 0) return total;               // wave-uniform
    int off = base;
    for (int k = 0; k < w; ++k) off += sW[k];
    if (PART && (off >= to || off + cnt <= from)) return total;   // wave-uniform
    if (words) {
        // the lane's 16 cells are 4 runs of 4 consecutive cells; faces in
        // ascending id order within a round: by lane, cell, axis
        for (int e = 0; e < COMPACT_CELLS_PER_THREAD / 4; ++e) {
            const unsigned bits12 = (unsigned)(packed >> (12 * e)) & 0xfffu;
            const int n = __popc(bits12);
            int incl = n;
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(incl, o);
                if (lane >= o) incl += y;
            }
            const int tot = __shfl(incl, 63);
            if (tot == 0) continue;                               // wave-uniform
            int o = off + incl - n;
            const int f0 = (int)(3u * (wbase + 256u * e + 4u * lane));
            if (!PART || (off >= from && off + tot <= to)) {      // wave-uniform, as a rule true
                for (int q = 0; q < 12; ++q)
                    if (bits12 & (1u << q)) {
                        a.queue[o] = f0 + q;                      // 3 (c0 + b) + d = f0 + 3b + d
                        a.fslot[f0 + q] = o;
                        ++o;
                    }
            } else if (off < to && off + tot > from) {
                for (int q = 0; q < 12; ++q)
                    if (bits12 & (1u << q)) {
                        if (o >= from && o < to) {
                            a.queue[o] = f0 + q;
                            a.fslot[f0 + q] = o;
                        }
                        ++o;
                    }
            }
            off += tot;
        }
        return total;
    }
    const bool whole = !PART || (off >= from && off + cnt <= to);   // wave-uniform, as a rule true
    // byte path: faces in ascending id order: by cell, then by axis
    const uint64_t below = (1ull << lane) - 1ull;
    for (int e = 0; e < COMPACT_CELLS_PER_THREAD; ++e) {
        const unsigned bits = (unsigned)(packed >> (3 * e)) & 7u;
        const uint64_t b0 = __ballot(bits & 1u), b1 = __ballot(bits & 2u), b2 = __ballot(bits & 4u);
        if ((b0 | b1 | b2) == 0ull) continue;
        int o = off + __popcll(b0 & below) + __popcll(b1 & below) + __popcll(b2 & below);
        const int f0 = (int)(3u * (wbase + lane + 64u * e));
#pragma unroll
        for (int d = 0; d < 3; ++d)
            if (bits & (1u << d)) {
                if (whole || (o >= from && o < to)) {
                    a.queue[o] = f0 + d;
                    a.fslot[f0 + d] = o;
                }
                ++o;
            }
        off += __popcll(b0) + __popcll(b1) + __popcll(b2);
    }
    return total;
}

// The queue entries and face slots of a chunk.  The counts before it are
// added up once and carried through its compaction blocks, so that a rebuild
// costs what the grid's size does (summed anew for each compaction block they
// were 0.4 GB of reads at 384^3 and 34 GB at 2^29 cells): counts and queue
// of a moving interface 74 + 120 -> 79 + 39 us at 384^3 and 161 + 382 ->
// 159 + 83 us at 512^3, where a count, a scan and a scatter in launches of
// their own, with a block per compaction block, took 69 + 16 + 44 and 148 +
// 58 + 95 us.
__device__ __forceinline__ void scatter_chunk(const IfaceArgs& a, int chunk)
{
    if (a.blockcnt[chunk] == 0) return;           // block-uniform
    const int2 r = chunk_blocks(a, chunk);
    int base = count_prefix(a, chunk);
    for (int blk = r.x; blk < r.y; ++blk) {
        base += scatter_body(a, blk, base);
        __syncthreads();                          // its sums are read before they are written again
    }
}

// A rebuilt queue shared out over the launch that also solves it, in units of
// at most COMPACT_THREADS faces of one compaction block.  Launch block b takes
// the first unit of compaction block b, which as a rule holds all its faces;
// the further units, where there are any, are numbered through and start at
// the launch blocks without a compaction block.  (With a compaction block per
// launch block, whatever it holds, an interface along a layer of the grid, all
// of whose faces lie in a few compaction blocks, is few blocks' work: a flat
// surface across z beside a moving bubble took 371 us per step at 128^3 and
// 172 at 64^3; 300 and 100 in units, 304 and 150 with the queue in launches of
// its own.  A launch block per unit in the order of the queue, every block
// scanning the counts for its first one, took 1 us more of a launch where no
// compaction block has a second unit, and 4 us at 50x43x37; no units at all 1.5
// us less there, and 0.5 us less with a kept queue, for the shorter code.)
constexpr int UNIT_BLOCKS = 2 * COMPACT_THREADS;      // compaction blocks at most
static_assert(UNIT_BLOCKS <= COMPACT_CHUNKS, "a count per compaction block");

// Units after the first of a compaction block of cnt faces.
__device__ __forceinline__ int further_units(int cnt) { return max(cnt - 1, 0) / COMPACT_THREADS; }

struct QueueShare {
    int base, cnt;                    // of the block's own compaction block: faces before it, and its faces
    int faces, further;               // of the whole queue: faces, and further units
    int c0, c1;                       // faces of compaction blocks 2t and 2t + 1, t the thread
};

__device__ __forceinline__ QueueShare queue_share(const IfaceArgs& a, int blk)
{
    __shared__ int sS[3][COMPACT_THREADS / 64];
    QueueShare u = {};
    const int b0 = 2 * (int)threadIdx.x;
    if (blk < a.nblk) u.cnt = a.blockcnt[blk];
    if (b0 < a.nblk) u.c0 = a.blockcnt[b0];
    if (b0 + 1 < a.nblk) u.c1 = a.blockcnt[b0 + 1];
    u.faces = u.c0 + u.c1;
    u.base = (b0 < blk ? u.c0 : 0) + (b0 + 1 < blk ? u.c1 : 0);
    u.further = further_units(u.c0) + further_units(u.c1);
    for (int o = 32; o > 0; o >>= 1) {
        u.faces += __shfl_xor(u.faces, o);
        u.base += __shfl_xor(u.base, o);
        u.further += __shfl_xor(u.further, o);
    }
    if ((threadIdx.x & 63) == 0) {
        sS[0][threadIdx.x >> 6] = u.faces;
        sS[1][threadIdx.x >> 6] = u.base;
        sS[2][threadIdx.x >> 6] = u.further;
    }
    __syncthreads();
    u.faces = u.base = u.further = 0;
    for (int k = 0; k < COMPACT_THREADS / 64; ++k) {
        u.faces += sS[0][k];
        u.base += sS[1][k];
        u.further += sS[2][k];
    }
    return u;
}

// Compaction block (x), its first queue position (y) and the positions [z, w)
// of further unit n.
__device__ __forceinline__ int4 find_unit(const QueueShare& qs, int n)
{
    __shared__ int sF[COMPACT_THREADS / 64], sU[COMPACT_THREADS / 64];
    __shared__ int4 sAt;
    const int b0 = 2 * (int)threadIdx.x, lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int c0 = qs.c0, c1 = qs.c1;
    const int f = c0 + c1, u = further_units(c0) + further_units(c1);
    int face = f, unit = u;
    for (int o = 1; o < 64; o <<= 1) {
        const int x = __shfl_up(face, o), y = __shfl_up(unit, o);
        if (lane >= o) {
            face += x;
            unit += y;
        }
    }
    if (lane == 63) {
        sF[w] = face;
        sU[w] = unit;
    }
    __syncthreads();
    face -= f;
    unit -= u;
    for (int k = 0; k < w; ++k) {
        face += sF[k];
        unit += sU[k];
    }
    int part = n - unit;
    if (part >= 0 && part < u) {                                  // one thread of the block
        const bool second = part >= further_units(c0);
        if (second) {
            part -= further_units(c0);
            face += c0;
        }
        const int from = face + (part + 1) * COMPACT_THREADS;
        sAt = make_int4(b0 + (second ? 1 : 0), face, from, min(from + COMPACT_THREADS, face + (second ? c1 : c0)));
    }
    __syncthreads();
    return sAt;
}

// The queue alone, and the opening of the step: where FIVER does not do both
// (fiver_opens), and listing the interface faces between steps.
__global__ __launch_bounds__(COMPACT_THREADS) void k_scatter(const IfaceArgs a, const StepOpen o)
{
    const bool reuse = a.sc->qreuse;
    if (blockIdx.x == 0) open_step(a, o, reuse ? 0 : count_total(a));
    if (!reuse) scatter_chunk(a, blockIdx.x);
}

hipError_t launch_scatter(const IfaceArgs& a, const StepOpen& o, hipStream_t s)
{
    hipLaunchKernelGGL(k_scatter, dim3(compact_chunks(a.nblk)), dim3(COMPACT_THREADS), 0, s, a, o);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// FIVER: one thread per queued face.  The Riemann data are the two cells'
// own (first-order) primitive states in the face frame (rho, u_n, p); the
// star states W*_L = (rho*_L, u*, tangential V_L, p*) and W*_R likewise feed
//   F_lower = HLLC(W_L, W*_L; EOS of the lower cell)
//   F_upper = HLLC(W*_R, W_R; EOS of the upper cell)
// with the arguments ordered along the face normal.
// FS: the set of the materials' families (EG; eos::fam_set)
template <bool EG, int FS = eos::FAM_ALL>
__device__ __forceinline__ void cell_prim(const Grid& G, const eos::EosK* sEos, const double* __restrict__ W,
                                          uint32_t c, int x, double q[5])
{
    const uint32_t N = (uint32_t)G.N;
    double u, v, w;
    if constexpr (EG)
        q[4] = geos_prim<FS>(sEos[x], ldf(W, c), ldf(W + N, c), ldf(W + 2 * N, c), ldf(W + 3 * N, c),
                             ldf(W + 4 * N, c), u, v, w);
    else
        q[4] = eos_prim(ldf(W, c), ldf(W + N, c), ldf(W + 2 * N, c), ldf(W + 3 * N, c), ldf(W + 4 * N, c),
                        pick(G.gamma, x) - 1.0, pick(G.gpc, x), u, v, w);
    q[0] = ldf(W, c);
    q[1] = u;
    q[2] = v;
    q[3] = w;
}

// EG: general EOS per material (the Riemann solve of section "Equations of
// state" with Hugoniot and isentrope wave curves, fluxes with each side's
// EOS).  LG: learned star-pressure guess (stiffened gases): each face first
// takes the near-equilibrium test, and only a wavefront holding a face that
// fails it loads the network and evaluates it (on the matrix cores, 64 faces
// per pass); every other face starts Newton from the acoustic guess at no
// extra cost.  The queue is then walked in whole wavefronts, since the
// network needs every lane of one; its operands are read from memory as
// they are needed, so that the kernel keeps the acoustic kernel's registers.
// F0, F1 (EG): families of materials 0 and 1 fixed at compile time, so that
// a kernel carries the wave curves and EOS forms of those two families only
// (-1: dispatched at run time).
// OPEN: the first launch of a step, which opens it (open) and writes a rebuilt
// queue: each block writes and solves units of it (queue_share; a unit is
// seldom full, as the interface lies in the grid, which costs little for
// stiffened gases, and saves a launch).
template <bool EG, bool LG = false, int F0 = -1, int F1 = -1, bool OPEN = false>
__device__ __forceinline__ void fiver_body(const IfaceArgs& a, int record, int blk, int nblk,
                                           const MlpDev* m = nullptr, const StepOpen* open = nullptr)
{
    static_assert(!OPEN || (!EG && !LG), "stiffened gases and the acoustic start open steps");
    static_assert(!(EG && LG) || (F0 >= 0 && F1 >= 0), "the general-EOS learned start needs the families");
    __shared__ unsigned long long sCnt[3][4];
    __shared__ int sHead[2];
    __shared__ eos::EosK sEos[EG ? 2 : 1];
    DevScalars* sc = a.sc;
    const Grid& G = a.g;
    constexpr int FS = eos::fam_set(F0) | eos::fam_set(F1);
    // nothing to do when an earlier kernel failed; read once per block so that
    // the whole block takes the same branch (this kernel's own reports may
    // raise the flag meanwhile; an opening launch's do not stop its blocks,
    // so that the queue they write between them is whole)
    const int q0 = blk * (int)blockDim.x + (int)threadIdx.x;
    // the thread's first entry of a kept queue, read beside the scalars that
    // say whether it counts (each dependent read is about 0.7 us of a launch
    // that takes 8 for a single face)
    const int32_t ahead = q0 < a.qcap ? a.queue[q0] : 0;
    if (threadIdx.x == 0) {
        const int err = sc->err, qlen = sc->qlen, reuse = sc->qreuse;
        sHead[0] = (OPEN ? failed_before(err) : err != 0) ? 0 : (OPEN && !reuse ? 1 : qlen);
        sHead[1] = OPEN && !reuse;
    }
    if (EG) geos_stage(G, sEos);
    else __syncthreads();
    const bool rebuilt = OPEN && sHead[1];
    const int n = sHead[0];
    QueueShare qs = {};
    if (rebuilt) {                                                   // block-uniform
        qs = queue_share(a, blk);
        // (no face of a queue past its capacity is solved: the overflow is
        // the step's one error, whichever block is first)
        if (n == 0 || qs.faces > a.qcap) qs.cnt = qs.further = 0;
    }
    if (OPEN && blk == 0) open_step(a, *open, qs.faces);
    long long iters = 0, fallbacks = 0, mlp_fb = 0;
    // A kept queue in one sweep of the launch, a rebuilt one unit by unit.
    // (Whole wavefronts of 64 faces and whole blocks first: a short queue
    // spread over more wavefronts at 8 faces each took longer: 128^3 charge
    // 87 -> 328 us, 50x43x37 9.5 -> 15.8 us.)
    const int known = rebuilt ? -1 : q0;
    // one queue entry per thread, the last wavefront's beyond the end not live
    auto face = [&](int q, bool live) __attribute__((always_inline)) {
        uint32_t c = 0, cn = 0;
        int d = 0;
        if (live) face_cells(G.nx, G.ny, G.nz, (uint32_t)(q == known ? ahead : a.queue[q]), c, cn, d);
        const int xa = live ? a.chi[c] : 0, xb = live ? a.chi[cn] : 0;
        double qa[5], qb[5];
        cell_prim<EG, FS>(G, sEos, a.Win, c, xa, qa);
        cell_prim<EG, FS>(G, sEos, a.Win, cn, xb, qb);
        const int t1 = 1 + (d + 1) % 3, t2 = 1 + (d + 2) % 3;
        const double ua = qa[1 + d], ub = qb[1 + d];
        const double gA = pick(G.gamma, xa), pcA = pick(G.pc, xa), gB = pick(G.gamma, xb), pcB = pick(G.pc, xb);
        double out[4];
        bool used = false;
        bool hg = false;
        double gs = 0.0;
        if constexpr (LG && !EG) {
            const bool skip = !live || acoustic_suffices(qa[0], ua, qa[4], gA, pcA, qb[0], ub, qb[4], gB, pcB);
            if (__ballot(!skip) != 0ull) {                       // wave-uniform
                float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                double plo = 0.0, P = 1.0;
                if (!skip) mlp_features(qa[0], ua, qa[4], gA, pcA, qb[0], ub, qb[4], gB, pcB, x, plo, P);
                gs = guess64_mem(*m, x, plo, P, skip);
                hg = !skip;
            }
            if (!live) return;
        }
        int it;
        if constexpr (EG) {
            // material 0 always on the left: where the lower cell holds
            // material 1 the mirrored problem is solved (p* unchanged, u*
            // negated, the star densities swapped), so that every lane of a
            // wavefront runs the same families' code on each side
            const bool flip = xa != 0;
            const double in[6] = {flip ? qb[0] : qa[0], flip ? -ub : ua, flip ? qb[4] : qa[4],
                                  flip ? qa[0] : qb[0], flip ? -ua : ub, flip ? qa[4] : qb[4]};
            double o[4];
            constexpr int S0 = eos::fam_set(F0), S1 = eos::fam_set(F1);
            if constexpr (LG) {
                // learned start (the families take it, see learned_pair):
                // the network evaluated by whole wavefronts for the faces
                // away from equilibrium, then the judged outer iteration
                eos::Pair P;
                const bool ok = live && eos::pair_init<S0, S1>(sEos[0], sEos[1], in, P);
                float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
                double plo = 0.0, Pn = 1.0;
                const bool skip = !ok || eos_near_equilibrium(P) || !eos_features(P, F0, F1, x, plo, Pn);
                double g = __builtin_nan("");
                if (__ballot(!skip) != 0ull) g = guess64_mem(*m, x, plo, Pn, skip);      // wave-uniform
                if (!live) return;
                it = 0;
                for (int k = 0; k < 4; ++k) o[k] = __builtin_nan("");
                if (ok) it = eos::pair_solve<S0, S1, 8>(sEos[0], sEos[1], P, G.rtol, G.maxit, G.rds, g, o, &used);
            } else {
                it = eos::solve_pair<S0, S1, 8>(sEos[0], sEos[1], in, G.rtol, G.maxit, G.rds, o);
            }
            out[0] = o[0];
            out[1] = flip ? -o[1] : o[1];
            out[2] = flip ? o[3] : o[2];
            out[3] = flip ? o[2] : o[3];
        } else {
            it = riemann_solve(qa[0], ua, qa[4], gA, pcA, qb[0], ub, qb[4], gB, pcB, G.rtol, G.maxit, hg, gs, out,
                               &used);
        }
        // faces that started from the acoustic guess (near equilibrium, or
        // the judge preferred it)
        mlp_fb += LG && !used && it != 0;
        if (it == 0) {
            report_error(&sc->err, &sc->err_cell, OPEN ? ST_RIEMANN_OPENING : ST_RIEMANN, c);
            return;
        }
        iters += it < 0 ? -it : it;
        fallbacks += it < 0;
        const double ps = out[0], us = out[1];
        double Fl[5], Fu[5];
        if constexpr (EG) {
            geos_flux<FS>(sEos[xa], G.flux, qa[0], ua, qa[t1], qa[t2], qa[4], out[2], us, qa[t1], qa[t2], ps, Fl);
            geos_flux<FS>(sEos[xb], G.flux, out[3], us, qb[t1], qb[t2], ps, qb[0], ub, qb[t1], qb[t2], qb[4], Fu);
        } else {
            num_flux<double>(G.flux, qa[0], ua, qa[t1], qa[t2], qa[4], out[2], us, qa[t1], qa[t2], ps, gA, pcA,
                             pick(G.gpc, xa), pick(G.inv_gm1, xa), Fl);
            num_flux<double>(G.flux, out[3], us, qb[t1], qb[t2], ps, qb[0], ub, qb[t1], qb[t2], qb[4], gB, pcB,
                             pick(G.gpc, xb), pick(G.inv_gm1, xb), Fu);
        }
        // face frame (mass, normal, t1, t2, energy) -> global components;
        // the ten fluxes of a face are contiguous (one address per face for
        // the stage kernel that reads them)
        double* const fq = a.fluxF + 10 * (long long)q;
        double fo[10];
        fo[0] = Fl[0];
        fo[1 + d] = Fl[1];
        fo[t1] = Fl[2];
        fo[t2] = Fl[3];
        fo[4] = Fl[4];
        fo[5] = Fu[0];
        fo[6 + d] = Fu[1];
        fo[5 + t1] = Fu[2];
        fo[5 + t2] = Fu[3];
        fo[9] = Fu[4];
#pragma unroll
        for (int v = 0; v < 10; ++v) fq[v] = fo[v];
        if (record) {
            const long long Q = a.qcap;
            a.star[0 * Q + q] = ps;
            a.star[1 * Q + q] = us;
            a.star[2 * Q + q] = out[2];
            a.star[3 * Q + q] = out[3];
            a.star[4 * Q + q] = qa[t1];
            a.star[5 * Q + q] = qa[t2];
            a.star[6 * Q + q] = qb[t1];
            a.star[7 * Q + q] = qb[t2];
        }
    };
    if constexpr (OPEN) {
        // (passes of a kept queue and units of a rebuilt one in one loop, so
        // that the solve is there once)
        int pass = rebuilt && blk < a.nblk && qs.cnt == 0 ? blk + nblk : blk;
        // (the launch has a.nblk blocks or more)
        // (block-uniform)
        while (rebuilt ? pass < a.nblk || pass - a.nblk < qs.further : pass * COMPACT_THREADS < n) {
            int from = pass * COMPACT_THREADS, to = n;
            if (rebuilt) {
                int4 at = make_int4(pass, qs.base, qs.base, qs.base + min(qs.cnt, COMPACT_THREADS));
                if (pass >= a.nblk) at = find_unit(qs, pass - a.nblk);
                from = at.z;
                to = at.w;
                scatter_body<true>(a, at.x, at.y, from, to);
                __syncthreads();                                     // the block reads its own entries
            }
            const int q = from + (int)threadIdx.x;
            if (q < to) face(q, true);
            pass += nblk;
        }
    } else {
        // LG: wave-uniform trip count (q may pass n in the last pass)
        const int qend = LG ? (n + 63) / 64 * 64 : n, stride = nblk * (int)blockDim.x;
        for (int q = q0; q < qend; q += stride) face(q, !LG || q < n);
    }
    // counters: one atomic per block and counter (same-address atomics from
    // every wavefront serialise into a measurable tail)
    for (int o = 32; o > 0; o >>= 1) {
        iters += __shfl_xor(iters, o);
        fallbacks += __shfl_xor(fallbacks, o);
        mlp_fb += __shfl_xor(mlp_fb, o);
    }
    const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        sCnt[0][w] = iters;
        sCnt[1][w] = fallbacks;
        sCnt[2][w] = mlp_fb;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        unsigned long long t = 0;
        for (int k = 0; k < nw; ++k) t += sCnt[threadIdx.x][k];
        unsigned long long* dst = threadIdx.x == 0 ? (unsigned long long*)&sc->newton_iters
                                 : (threadIdx.x == 1 ? (unsigned long long*)&sc->fallbacks
                                                     : (unsigned long long*)&sc->mlp_fallbacks);
        if (t) atomicAdd(dst, t);
    }
}

static_assert(COMPACT_THREADS == 256, "the FIVER kernels run compaction blocks");

__global__ __launch_bounds__(256) void k_fiver(const IfaceArgs a, int record)
{
    fiver_body<false>(a, record, blockIdx.x, gridDim.x);
}

__global__ __launch_bounds__(256) void k_fiver_open(const IfaceArgs a, int record, const StepOpen o)
{
    fiver_body<false, false, -1, -1, true>(a, record, blockIdx.x, gridDim.x, nullptr, &o);
}

template <int F0, int F1>
__global__ __launch_bounds__(256) void k_fiver_eos(const IfaceArgs a, int record)
{
    fiver_body<true, false, F0, F1>(a, record, blockIdx.x, gridDim.x);
}

// with the learned start, for the family pairs that take it (learned_pair)
template <int F0, int F1>
__global__ __launch_bounds__(256) void k_fiver_eos_learned(const IfaceArgs a, int record, const MlpDev m)
{
    fiver_body<true, true, F0, F1>(a, record, blockIdx.x, gridDim.x, &m);
}

template <int F0, int F1>
void launch_fiver_eos(const IfaceArgs& a, unsigned nb, int record, const MlpDev* mlp, hipStream_t s)
{
    if constexpr (learned_pair(F0, F1)) {
        if (mlp) {
            hipLaunchKernelGGL((k_fiver_eos_learned<F0, F1>), dim3(nb), dim3(256), 0, s, a, record, *mlp);
            return;
        }
    }
    hipLaunchKernelGGL((k_fiver_eos<F0, F1>), dim3(nb), dim3(256), 0, s, a, record);
}
using FiverEosLaunch = void (*)(const IfaceArgs&, unsigned, int, const MlpDev*, hipStream_t);
// by 3 family(material 0) + family(material 1), families NASG, MG, JWL = 0, 1, 2
constexpr FiverEosLaunch kFiverEos[9] = {launch_fiver_eos<0, 0>, launch_fiver_eos<0, 1>, launch_fiver_eos<0, 2>,
                                         launch_fiver_eos<1, 0>, launch_fiver_eos<1, 1>, launch_fiver_eos<1, 2>,
                                         launch_fiver_eos<2, 0>, launch_fiver_eos<2, 1>, launch_fiver_eos<2, 2>};
static_assert(M2C_EOS_NASG == 0 && M2C_EOS_MG == 1 && M2C_EOS_JWL == 2, "family-pair table order");

__global__ __launch_bounds__(256) void k_fiver_learned(const IfaceArgs a, int record, const MlpDev m)
{
    fiver_body<false, true>(a, record, blockIdx.x, gridDim.x, &m);
}

// With a general EOS the queue is a launch of its own: a face takes so long
// there that spreading the faces as the interface lies in the grid costs more
// than the launch (128^3 charge, a compaction block to a launch block: FIVER 80
// -> 131 us); with the learned guess too, whose network takes whole wavefronts
// of faces; and on grids of more compaction blocks than a launch block looks
// after counts (queue_share), where the queue is work, not latency (384^3, a
// compaction block to a launch block: the first FIVER launch 64 us against 30,
// of a 5 ms step).
bool fiver_opens(const IfaceArgs& a, const MlpDev* mlp) { return !(a.g.eosg || mlp || a.nblk > UNIT_BLOCKS); }

hipError_t launch_fiver(const IfaceArgs& a, bool record, const StepOpen* open, const MlpDev* mlp, hipStream_t s)
{
    if (open && !fiver_opens(a, mlp)) return hipErrorInvalidValue;
    long long nb = (a.qcap + 255) / 256;
    if (nb > 1024) nb = 1024;
    if (nb < 1) nb = 1;
    const int rec = record ? 1 : 0;
    if (a.g.eosg) {
        const int f0 = a.g.ek[0].fam, f1 = a.g.ek[1].fam;
        if (f0 < 0 || f0 > 2 || f1 < 0 || f1 > 2) return hipErrorInvalidValue;
        kFiverEos[3 * f0 + f1](a, (unsigned)nb, rec, mlp, s);
    } else if (mlp) {
        hipLaunchKernelGGL(k_fiver_learned, dim3((unsigned)nb), dim3(256), 0, s, a, rec, *mlp);
    } else if (open) {
        // a rebuilt queue takes a block per compaction block
        if (nb < a.nblk) nb = a.nblk;
        hipLaunchKernelGGL(k_fiver_open, dim3((unsigned)nb), dim3(256), 0, s, a, rec, *open);
    } else {
        hipLaunchKernelGGL(k_fiver, dim3((unsigned)nb), dim3(256), 0, s, a, rec);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Phase update (step 6 of the time-step outline, section "Code structure"):
// material ids follow the sign of the new level set; a cell that changed
// from material A to B takes the mean, over its faces in the order
// -x,+x,-y,+y,-z,+z whose neighbour held B during the step, of the B-side
// star state of the last stage's Riemann problem there (rho*_B, the B
// cell's velocity with its normal component replaced by u*, p*), encoded
// with B's equation of state.  Without such a face it keeps its primitive
// state (an "orphan").  The new state also enters the next step's CFL
// maximum.
template <bool EG>
__device__ __forceinline__ void phase_body(const PhaseArgs& a, int blk, int nblk)
{
    DevScalars* sc = a.sc;
    const Grid& G = a.g;
    __shared__ eos::EosK sEos[EG ? 2 : 1];
    if constexpr (EG) geos_stage(G, sEos);
    if (sc->err != 0) return;
    const int n = sc->nflip;
    const long long N = G.N, sxy = (long long)G.nx * G.ny, Q = a.qcap;
    double lam = 0.0;
    long long orphans = 0;
    for (int e = blk * blockDim.x + threadIdx.x; e < n; e += nblk * blockDim.x) {
        const long long c = a.flips[e];
        const int A = a.chi_old[c], B = a.chi_new[c];
        // (32-bit: grids hold at most 2^29 cells)
        const uint32_t c32 = (uint32_t)c, pl = (uint32_t)sxy;
        const int k = (int)(c32 / pl);
        const uint32_t r = c32 - (uint32_t)k * pl;
        const int j = (int)(r / (uint32_t)G.nx);
        const int i = (int)(r - (uint32_t)j * (uint32_t)G.nx);
        // the six faces side by side: neighbours' ids, then the queue slots
        // of the faces whose neighbour held B, then their star states (three
        // memory latencies instead of three per face); summed in the order
        // of the faces
        long long lower[6];
        bool held[6];
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const int d = f / 2, side = f % 2;
            const int nd = d == 0 ? G.nx : (d == 1 ? G.ny : G.nz), at = d == 0 ? i : (d == 1 ? j : k);
            const long long str = d == 0 ? 1 : (d == 1 ? (long long)G.nx : sxy);
            int nb = at + (side ? 1 : -1);
            const bool out = nb < 0 || nb >= nd;
            if (out) nb = side ? 0 : nd - 1;
            const bool face = G.act[d] && (!out || G.bc[f] == BC_PERIODIC);
            const long long ck = face ? c + (long long)(nb - at) * str : c;
            lower[f] = side ? c : ck;
            held[f] = face && a.chi_old[ck] == B;
        }
        int sl[6];
#pragma unroll
        for (int f = 0; f < 6; ++f) sl[f] = held[f] ? a.fslot[3 * lower[f] + f / 2] : -1;
        double st[6][5];
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const int side = f % 2;
            if (sl[f] >= 0) {
                st[f][0] = a.star[(side ? 3 : 2) * Q + sl[f]];
                st[f][1] = a.star[1 * Q + sl[f]];
                st[f][2] = a.star[(side ? 6 : 4) * Q + sl[f]];
                st[f][3] = a.star[(side ? 7 : 5) * Q + sl[f]];
                st[f][4] = a.star[0 * Q + sl[f]];
            }
        }
        double sum[5] = {0, 0, 0, 0, 0};
        int cnt = 0;
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const int d = f / 2, t1 = 1 + (d + 1) % 3, t2 = 1 + (d + 2) % 3;
            if (sl[f] >= 0) {
                sum[0] += st[f][0];
                sum[1 + d] += st[f][1];
                sum[t1] += st[f][2];
                sum[t2] += st[f][3];
                sum[4] += st[f][4];
                ++cnt;
            }
        }
        double q[5];
        if (cnt) {
#pragma unroll
            for (int v = 0; v < 5; ++v) q[v] = sum[v] / cnt;
        } else {
            double u, vv, w;
            if constexpr (EG)
                q[4] = geos_prim(sEos[A], a.W[c], a.W[N + c], a.W[2 * N + c], a.W[3 * N + c], a.W[4 * N + c], u, vv, w);
            else
                q[4] = eos_prim(a.W[c], a.W[N + c], a.W[2 * N + c], a.W[3 * N + c], a.W[4 * N + c],
                                pick(G.gamma, A) - 1.0, pick(G.gpc, A), u, vv, w);
            q[0] = a.W[c];
            q[1] = u;
            q[2] = vv;
            q[3] = w;
            ++orphans;
        }
        bool ok = EG ? geos_ok(sEos[B], q[0], q[4]) : q[0] > 0.0 && q[4] + pick(G.pc, B) > 0.0;
#pragma unroll
        for (int v = 0; v < 5; ++v) ok = ok && isfinite(q[v]);
        if (!ok) report_error(&sc->err, &sc->err_cell, ST_NONPHYSICAL, c);
        a.W[c] = q[0];
        a.W[N + c] = q[0] * q[1];
        a.W[2 * N + c] = q[0] * q[2];
        a.W[3 * N + c] = q[0] * q[3];
        if constexpr (EG) a.W[4 * N + c] = geos_energy(sEos[B], q[0], q[1], q[2], q[3], q[4]);
        else a.W[4 * N + c] = eos_energy<double>(q[0], q[1], q[2], q[3], q[4], pick(G.gpc, B), pick(G.inv_gm1, B));
        if (ok) {
            const double cs = EG ? sqrt(geos_c2(sEos[B], q[0], q[4])) : sqrt(pick(G.gamma, B) * (q[4] + pick(G.pc, B)) / q[0]);
            double l = 0.0;
            for (int d = 0; d < 3; ++d)
                if (G.act[d]) l += (fabs(q[1 + d]) + cs) * G.rh[d];
            lam = fmax(lam, l);
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        lam = fmax(lam, __shfl_xor(lam, o));
        orphans += __shfl_xor(orphans, o);
    }
    if ((threadIdx.x & 63) == 0) {
        if (lam > 0.0) atomic_max_nonneg(&sc->lam_bits, lam);
        if (orphans) atomicAdd((unsigned long long*)&sc->orphans, (unsigned long long)orphans);
    }
}

__global__ __launch_bounds__(256) void k_phase(const PhaseArgs a) { phase_body<false>(a, blockIdx.x, gridDim.x); }
__global__ __launch_bounds__(256) void k_phase_eos(const PhaseArgs a) { phase_body<true>(a, blockIdx.x, gridDim.x); }

hipError_t launch_phase(const PhaseArgs& a, hipStream_t s)
{
    long long nb = (a.g.N + 255) / 256;
    if (nb > 256) nb = 256;
    if (a.g.eosg)
        hipLaunchKernelGGL(k_phase_eos, dim3((unsigned)nb), dim3(256), 0, s, a);
    else
        hipLaunchKernelGGL(k_phase, dim3((unsigned)nb), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Start of a single-grid step: the phase update of the previous step of the
// same m2c_step call (prev: it writes the state at flipped cells, the CFL
// maximum and error reports) and the count of interface faces per block
// (reads only material ids), neither where the queue is kept.  The launch
// after it opens the step (open_step).
template <bool EG>
__global__ __launch_bounds__(COMPACT_THREADS) void k_step_begin(const IfaceArgs a, const PhaseArgs pa, int prev)
{
    const int err = a.sc->err;                    // (read beside the words of the decision)
    const bool kept = queue_kept(a.sc);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.sc->qreuse = kept ? 1 : 0;
        settle_error(a.sc, err);                  // (stays an error to the blocks that read it meanwhile)
    }
    if (kept) return;
    if (prev) phase_body<EG>(pa, blockIdx.x, gridDim.x);
    count_body(a, blockIdx.x);
}

hipError_t launch_step_begin(const IfaceArgs& a, const PhaseArgs* prev_phase, hipStream_t s)
{
    const PhaseArgs pa = prev_phase ? *prev_phase : PhaseArgs{};
    const int prev = prev_phase ? 1 : 0;
    if (prev_phase && a.g.eosg)
        hipLaunchKernelGGL(k_step_begin<true>, dim3(compact_chunks(a.nblk)), dim3(COMPACT_THREADS), 0, s, a, pa, prev);
    else
        hipLaunchKernelGGL(k_step_begin<false>, dim3(compact_chunks(a.nblk)), dim3(COMPACT_THREADS), 0, s, a, pa, prev);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Batched forms: the same bodies over many independent runs.  Each run's
// arguments are rebuilt on the device from its descriptor and its
// device-side state parity (sc->cur), so a captured graph is valid for
// every step.
__device__ __forceinline__ IfaceArgs iface_of_run(const RunDesc& R, int stage)
{
    IfaceArgs a;
    const int cur = R.sc->cur;
    a.g = R.g;
    a.Win = stage == 2 ? R.W1 : R.W[cur];
    a.chi = R.chi[cur];
    a.queue = R.queue;
    a.fslot = R.fslot;
    a.fluxF = R.fluxF;
    a.star = R.star;
    a.blockcnt = R.blockcnt;
    a.qcap = R.qcap;
    a.nblk = R.nblk_compact;
    a.sc = R.sc;
    return a;
}

// The two launches that start a batch step, as for a single grid: the counts
// of the runs whose queue is not kept; then the opening of every run's step
// and the queues.  (The phase update and the end of the step before, which
// turns the state parity, are launches of their own.)
__global__ __launch_bounds__(COMPACT_THREADS) void k_count_batch(const RunDesc* __restrict__ runs,
                                                                 const int2* __restrict__ cmap)
{
    const int2 m = cmap[blockIdx.x];
    DevScalars* sc = runs[m.x].sc;
    const bool kept = queue_kept(sc);
    if (m.y == 0 && threadIdx.x == 0) sc->qreuse = kept ? 1 : 0;
    if (kept) return;
    count_body(iface_of_run(runs[m.x], 1), m.y);
}

__global__ __launch_bounds__(COMPACT_THREADS) void k_scatter_batch(const RunDesc* __restrict__ runs,
                                                                   const int2* __restrict__ cmap)
{
    const int2 m = cmap[blockIdx.x];
    const bool reuse = runs[m.x].sc->qreuse;
    if (reuse && m.y != 0) return;
    const IfaceArgs a = iface_of_run(runs[m.x], 1);
    if (m.y == 0) open_step(a, StepOpen{0, 1, 0.0}, reuse ? 0 : count_total(a));
    if (!reuse) scatter_chunk(a, m.y);
}

hipError_t launch_compact_batch(const RunDesc* runs, const int2* cmap, int ncblocks, hipStream_t s)
{
    hipLaunchKernelGGL(k_count_batch, dim3(ncblocks), dim3(COMPACT_THREADS), 0, s, runs, cmap);
    hipLaunchKernelGGL(k_scatter_batch, dim3(ncblocks), dim3(COMPACT_THREADS), 0, s, runs, cmap);
    return hipGetLastError();
}

__global__ __launch_bounds__(64) void k_fiver_batch(const RunDesc* __restrict__ runs, int stage, int per_run)
{
    const int r = blockIdx.x / per_run, b = blockIdx.x % per_run;
    fiver_body<false>(iface_of_run(runs[r], stage), stage == 2, b, per_run);
}

// One-wavefront blocks, about 8192 over the batch (the solves
// of a run in one or two passes), between 32 and 256 per run (a 128^3 bubble
// of radius 0.25 has 19000 faces).  16 runs of edges 32..128: 33.7 us at 32
// per run, 19 at 256.
hipError_t launch_fiver_batch(const RunDesc* runs, int nruns, int stage, hipStream_t s)
{
    int per = 8192 / nruns;
    per = per < 32 ? 32 : (per > 256 ? 256 : per);
    hipLaunchKernelGGL(k_fiver_batch, dim3((unsigned)(nruns * per)), dim3(64), 0, s, runs, stage, per);
    return hipGetLastError();
}

constexpr int PHASE_BLOCKS_PER_RUN = 8;

__global__ __launch_bounds__(256) void k_phase_batch(const RunDesc* __restrict__ runs)
{
    const int r = blockIdx.x / PHASE_BLOCKS_PER_RUN, b = blockIdx.x % PHASE_BLOCKS_PER_RUN;
    const RunDesc& R = runs[r];
    const int cur = R.sc->cur;
    PhaseArgs a;
    a.g = R.g;
    a.W = R.W[cur ^ 1];
    a.chi_old = R.chi[cur];
    a.chi_new = R.chi[cur ^ 1];
    a.flips = R.flips;
    a.fslot = R.fslot;
    a.star = R.star;
    a.qcap = R.qcap;
    a.sc = R.sc;
    phase_body<false>(a, b, PHASE_BLOCKS_PER_RUN);
}

hipError_t launch_phase_batch(const RunDesc* runs, int nruns, hipStream_t s)
{
    hipLaunchKernelGGL(k_phase_batch, dim3(nruns * PHASE_BLOCKS_PER_RUN), dim3(256), 0, s, runs);
    return hipGetLastError();
}

}  // namespace m2c

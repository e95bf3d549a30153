// Device parts of a list build, shared by the list kernels of a build
// outside a step (dem_lists.hip) and by the step kernels that carry a build
// inside a step (dem_force.hip, dem_integrate.hip):
//   * nbr_rows: the neighbour rows of 4 particles by one wavefront (16
//     lanes per particle);
//   * fill_part: the pair offsets and pair entries of a quarter of a chunk
//     by one wavefront;
//   * plan: the tile plan of the pair kernel by one workgroup.
// The list decisions are an integer contract: |minimum image (x_j -
// x_i)|^2 < r_list^2 evaluated in FP64 as written, with no contraction into
// fused multiply-adds (the pragma at the top of each function body that
// evaluates them).
#pragma once

#include "dem_internal.h"

namespace dem {
namespace lb {

constexpr int kNbrLanes = 16;                 // lanes per particle in nbr_rows
constexpr int kNbrPer = lb_rows_per_group;    // particles per nbr_rows wavefront
static_assert(kNbrPer * kNbrLanes == 64, "one wavefront per group of particles");
constexpr int kNb3 = 27;                      // neighbour cells, the own one included
constexpr int kCellQuads = kCellCap / 4;
static_assert(kCellCap % 4 == 0 && kRowMax % 4 == 0 && kNb3 * kCellCap <= 65536, "quads of slots, in 16 bits");

// LDS of an nbr_rows wavefront, per particle: its hits, its neighbour cells
// and their occupied slots, four to an entry.  Rows are read in 16-byte words.
struct alignas(16) RowBuf {
    int row[kNbrPer][kRowMax];
    int cell[kNbrPer][kNb3];
    unsigned short quad[kNbrPer][kNb3 * kCellQuads];  // (cell * kCellQuads + quad) * 4 + slots in use - 1
};
static_assert(alignof(RowBuf) % 16 == 0 && offsetof(RowBuf, row) % 16 == 0 && sizeof(RowBuf::row[0]) % 16 == 0,
              "every row starts on a 16-byte boundary, wherever the compiler puts the buffer");

// Minimum image of d = x_j - x_i for positions in [0, L].  This equals
// d - L rint(d / L) bit for bit except where |d| is within rounding of L/2,
// and there both forms give |d| >= L/2 >= r_list, so no list decision can
// differ; it avoids an FP64 division per candidate.
__device__ inline double min_image(double d, double L)
{
    const double h = 0.5 * L;
    return d > h ? d - L : (d < -h ? d + L : d);
}

__device__ inline bool within(const SysParams &p, const StatePtrs &s, double xi, double yi, double zi, int j)
{
#pragma clang fp contract(off)
    const double dx = min_image(s.x[j] - xi, p.box[0]);
    const double dy = min_image(s.y[j] - yi, p.box[1]);
    double r2 = dx * dx + dy * dy;
    if (p.dim == 3) {
        const double dz = min_image(s.z[j] - zi, p.box[2]);
        r2 = r2 + dz * dz;
    }
    return r2 < p.rl2;
}

__device__ inline unsigned long long lanes_below()
{
    const unsigned lane = __lane_id();
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// Does this build take replica r?  (LISTS_REFILL: every live replica that
// has lists; LISTS_STEP: a replica whose step rebuilds and has steps left,
// FLAG_BUILD.)
__device__ inline bool building(int mode, int r, const SysParams &p, const int32_t *fl)
{
    if (!p.live) return false;
    if (mode == LISTS_STEP) return fl[FLAG_BUILD] != 0;
    if (mode == LISTS_REFILL) return fl[FLAG_NBUILDS] > 0;
    return mode == LISTS_ALL || mode == r;
}

// Exclusive scan of count[0..m) into start[0..m) by one workgroup of NT
// threads (count may be start; it is read through volatile loads, as other
// workgroups wrote it); part holds NT ints of LDS.  Returns the total.
template <int NT>
__device__ int block_scan(const int32_t *count, int32_t *start, int m, int *part)
{
    const volatile int32_t *vc = count;
    const int t = threadIdx.x;
    const int per = (m + NT - 1) / NT;
    const int lo = min(t * per, m), hi = min(lo + per, m);
    int sum = 0;
    for (int c = lo; c < hi; ++c) sum += vc[c];
    part[t] = sum;
    __syncthreads();
    for (int off = 1; off < NT; off <<= 1) {
        const int v = (t >= off) ? part[t - off] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int run = part[t] - sum;
    for (int c = lo; c < hi; ++c) {
        const int cnt = vc[c];
        start[c] = run;
        run += cnt;
    }
    const int total = part[NT - 1];
    __syncthreads();
    return total;
}

// Orders a wavefront's LDS writes before its reads after this.
__device__ inline void rows_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Neighbour rows of particles 4 vb .. 4 vb + 3 (all of one chunk, so of one
// replica), by one wavefront (a workgroup of 64 threads; the caller has
// checked that the replica builds).  The occupied slots of a particle's
// neighbour cells are listed in LDS, four to an entry, and dealt over its 16
// lanes, so that each lane has four candidates' loads under way at once and
// all lanes end together (or, without cells, each lane scans a sixteenth of
// the replica); hits are appended to the particle's LDS buffer in ballot
// order, then every kept hit finds its rank (the number of smaller hits) and
// is stored in that row slot, so the row ascends and keeps the cap smallest
// j.  The row's count of j > i is the particle's pair count.  The wavefront
// adds its total to its chunk's (ListPtrs::ctot, cleared when the build
// starts), and the chunk's last adds the chunk's to the replica's
// FLAG_NEWPAIRS: one addition to that word per chunk.
//
// What bounds it is the chain of loads, cell count, slot, position.  With a
// cell per lane (27 over 16 lanes) and one candidate per lane under way, a
// rank search that read LDS a word at a time, a same-address addition per
// wavefront and neighbouring rows written by different XCDs, the rows of
// 32,768 octahedra (52 slots a row) took 128 us; they take 51.
template <int DIM>
__device__ void nbr_rows(const BatchParams &b, const SysParams &p, const StatePtrs &s, const ListPtrs &l, int32_t *fl,
                         int vb, RowBuf &buf)
{
    const int end = p.off + p.n;
    if (vb * kNbrPer >= end) return;
    const int g = threadIdx.x / kNbrLanes, sub = threadIdx.x % kNbrLanes;
    const int i = vb * kNbrPer + g;
    int *row = buf.row[g];
    const bool mine = i < end;
    const int self = mine ? i : p.off;
    const unsigned long long gmask = 0xffffull << (kNbrLanes * ((threadIdx.x & 63) / kNbrLanes));
    const unsigned long long below = lanes_below() & gmask;
    const double xi = s.x[self], yi = s.y[self], zi = DIM == 3 ? s.z[self] : 0.0;
    int m = 0;  // hits so far (the same in all lanes of the particle)
    if (p.use_cells) {
        const int c = l.pcell[self];
        const int cx = c % p.nc[0], cy = (c / p.nc[0]) % p.nc[1], cz = c / (p.nc[0] * p.nc[1]);
        constexpr int kNb = DIM == 3 ? kNb3 : 9;
        constexpr int kPass = (kNb + kNbrLanes - 1) / kNbrLanes;
        int cnt[kPass];
#pragma unroll
        for (int u = 0; u < kPass; ++u) {
            const int t = u * kNbrLanes + sub;
            cnt[u] = 0;
            if (mine && t < kNb) {
                int ax = cx + t % 3 - 1, ay = cy + (t / 3) % 3 - 1, az = cz + (DIM == 3 ? t / 9 - 1 : 0);
                ax += (ax < 0) ? p.nc[0] : 0;
                ax -= (ax >= p.nc[0]) ? p.nc[0] : 0;
                ay += (ay < 0) ? p.nc[1] : 0;
                ay -= (ay >= p.nc[1]) ? p.nc[1] : 0;
                az += (az < 0) ? p.nc[2] : 0;
                az -= (az >= p.nc[2]) ? p.nc[2] : 0;
                const int cc = p.coff + ax + p.nc[0] * (ay + p.nc[1] * az);
                buf.cell[g][t] = cc;
                cnt[u] = min(l.cell_count[cc], kCellCap);
            }
        }
        int nq = 0;  // entries listed
#pragma unroll
        for (int u = 0; u < kPass; ++u) {
            const int t = u * kNbrLanes + sub, q = (cnt[u] + 3) / 4;
            int incl = q;
            for (int off = 1; off < kNbrLanes; off <<= 1) {
                const int v = __shfl_up(incl, off, kNbrLanes);
                if (sub >= off) incl += v;
            }
            unsigned short *out = buf.quad[g] + nq + incl - q;
            for (int k = 0; k < q; ++k)
                out[k] = (unsigned short)((t * kCellQuads + k) * 4 + min(cnt[u] - 4 * k, 4) - 1);
            nq += __shfl(incl, kNbrLanes - 1, kNbrLanes);
        }
        rows_sync();
        for (int e = sub;; e += kNbrLanes) {
            const bool has = e < nq;
            if (__ballot(has) == 0) break;
            int4 j = make_int4(self, self, self, self);
            if (has) {
                const int code = buf.quad[g][e], n = code & 3, t = code / (4 * kCellQuads);
                const int4 w = *reinterpret_cast<const int4 *>(l.cell_slot + (size_t)buf.cell[g][t] * kCellCap +
                                                               ((code >> 2) & (kCellQuads - 1)) * 4);
                j.x = w.x;  // slots not in use hold anything
                j.y = n > 0 ? w.y : self;
                j.z = n > 1 ? w.z : self;
                j.w = n > 2 ? w.w : self;
            }
            const int js[4] = {j.x, j.y, j.z, j.w};
            bool hit[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) hit[u] = (int)(js[u] != self) & (int)within(p, s, xi, yi, zi, js[u]);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned long long hm = __ballot(hit[u]);
                const int pos = m + __popcll(hm & below);
                if (hit[u] && pos < kRowMax) row[pos] = js[u];
                m += __popcll(hm & gmask);
            }
        }
    } else {
        for (int k0 = 0; k0 < p.n; k0 += kNbrLanes) {
            const int j = p.off + k0 + sub;
            const bool hit = mine && k0 + sub < p.n && j != i && within(p, s, xi, yi, zi, j);
            const unsigned long long hm = __ballot(hit);
            const int pos = m + __popcll(hm & below);
            if (hit && pos < kRowMax) row[pos] = j;
            m += __popcll(hm & gmask);
        }
    }
    const size_t N = (size_t)b.N;
    const int cap = b.cap;
    const int mm = min(m, kRowMax), quads = (mm + 3) / 4;
    if (sub < 4 * quads - mm) row[mm + sub] = 0x7fffffff;
    rows_sync();
    int lower = 0;  // kept hits below i
    for (int e0 = 0; e0 < mm; e0 += 4 * kNbrLanes) {  // four hits per lane at a time
        int v[4], rank[4] = {0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * kNbrLanes + sub;
            v[u] = e < mm ? row[e] : -1;
        }
        for (int f = 0; f < quads; ++f) {
            const int4 w = reinterpret_cast<const int4 *>(row)[f];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                rank[u] += (int)(w.x < v[u]) + (int)(w.y < v[u]) + (int)(w.z < v[u]) + (int)(w.w < v[u]);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (mine && v[u] >= 0 && rank[u] < cap) {
                l.nbr[(size_t)rank[u] * N + i] = v[u];
                lower += v[u] < i ? 1 : 0;
            }
    }
    for (int off = kNbrLanes / 2; off > 0; off >>= 1) lower += __shfl_xor(lower, off, kNbrLanes);
    const int kept = min(m, cap);
    if (mine && sub == 0) {
        l.n_nbr[i] = kept;
        l.klo[i] = lower;
        if (m > cap) atomicMax(&fl[FLAG_MAXROW], m);
        l.xlast[i] = xi;
        l.xlast[N + i] = yi;
        l.xlast[2 * N + i] = zi;
    }
    // the wavefront's pair count (integer sums, in any order)
    int tot = (mine && sub == 0) ? kept - lower : 0;
    for (int off = 32; off > 0; off >>= 1) tot += __shfl_xor(tot, off, 64);
    if (threadIdx.x == 0) {
        const int c = vb * kNbrPer / kChunk;
        const int parts = (min(end - c * kChunk, kChunk) + kNbrPer - 1) / kNbrPer;  // wavefronts of this chunk
        const int sum = atomicAdd(&l.ctot[c], tot + kChunkPart) + tot;
        if (sum / kChunkPart == parts - 1) atomicAdd(&fl[FLAG_NEWPAIRS], sum % kChunkPart);
    }
    rows_sync();  // buf is free for the next call once every lane has read it
}

// Pair offsets (unless `refill`: the offsets are kept) and pair entries of
// the 16 particles of quarter `part` of chunk c of replica p, by one
// wavefront, then their cells emptied when `clear_cells`.  The offset of i
// is the counts of the replica's chunks (ctot) before this one plus the
// counts of the chunk's particles before i.  The owner i of pair q writes
// {i, j, slot of j in i's row, slot of i in j's row} with one store, the
// last found by bisection in j's row (-1 if a row overflow left i out of it,
// which is reported).
//
// What bounds it is the chain of loads of the bisections, so a particle's
// pairs are dealt over four lanes, and a lane searches for four at once
// (32,768 octahedra 13.5 us; a lane per particle, one pair at a time, 40).
constexpr int kFillLanes = 4, kFillPer = 64 / kFillLanes, kFillParts = kChunk / kFillPer, kFillPairs = 4;
__device__ inline void fill_part(const BatchParams &b, const SysParams &p, const ListPtrs &l, int c, int part,
                                 bool refill, bool clear_cells)
{
    const int lane = __lane_id(), sub = lane % kFillLanes;
    const int end = p.off + p.n;
    const int i = c * kChunk + part * kFillPer + lane / kFillLanes;
    const size_t N = (size_t)b.N;
    int start = 0;
    if (!refill) {
        const int t = c * kChunk + lane;
        const int cnt = t < end ? l.n_nbr[t] - l.klo[t] : 0;
        int prior = 0;
#pragma unroll 8
        for (int q = p.off / kChunk + lane; q < c; q += 64) prior += l.ctot[q] % kChunkPart;
        int incl = cnt;
        for (int off = 1; off < 64; off <<= 1) {
            const int v = __shfl_up(incl, off, 64);
            if (lane >= off) incl += v;
        }
        for (int off = 32; off > 0; off >>= 1) prior += __shfl_xor(prior, off, 64);
        start = __shfl(prior + incl - cnt, part * kFillPer + lane / kFillLanes, 64);
    }
    if (i >= end) return;
    if (refill) start = l.pstart[i];
    else if (sub == 0) l.pstart[i] = start;
    const int m = min(l.n_nbr[i], b.cap), k0 = max(l.klo[i], 0);
    int4 *pairs = l.pairs + p.poff;
    for (int kb = k0 + sub; kb < m; kb += kFillLanes * kFillPairs) {
        int j[kFillPairs], lo[kFillPairs], hi[kFillPairs], w[kFillPairs];
#pragma unroll
        for (int u = 0; u < kFillPairs; ++u) j[u] = l.nbr[(size_t)min(kb + u * kFillLanes, m - 1) * N + i];
#pragma unroll
        for (int u = 0; u < kFillPairs; ++u) {
            lo[u] = 0;
            hi[u] = l.klo[j[u]];  // j's neighbours below j, ascending
            w[u] = -1;
        }
        for (;;) {
            bool open = false;
            int v[kFillPairs];
#pragma unroll
            for (int u = 0; u < kFillPairs; ++u) {
                open |= lo[u] < hi[u];
                v[u] = l.nbr[(size_t)min((lo[u] + hi[u]) >> 1, b.cap - 1) * N + j[u]];
            }
            if (!open) break;
#pragma unroll
            for (int u = 0; u < kFillPairs; ++u) {
                const int mid = (lo[u] + hi[u]) >> 1;
                if (lo[u] < hi[u]) {
                    if (v[u] == i) w[u] = mid;
                    if (v[u] < i) lo[u] = mid + 1;
                    else hi[u] = mid;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kFillPairs; ++u) {
            const int k = kb + u * kFillLanes, q = start + (k - k0);
            // (q >= pcap only after a row overflow, which is reported)
            if (k < m && q < p.pcap) pairs[q] = make_int4(i, j[u], k, w[u]);
        }
    }
    // every particle of the cell writes the same zero (without cells the
    // word is zero already; use_cells of a replica under the barostat may
    // change while this runs)
    if (clear_cells && sub == 0) l.cell_count[p.coff + l.pcell[i]] = 0;
}

// Tile plan (the first tile of each replica, b.tile pairs per tile) by one
// workgroup of NT threads; a replica for which built(r) holds takes its new
// pair total (FLAG_NEWPAIRS) first.  part: NT ints of LDS.
template <int NT, typename Built>
__device__ void plan(const BatchParams &b, const SysParams *reps, const ListPtrs &l, int *part, Built built)
{
    const volatile int32_t *vfl = l.flags;
    for (int r = threadIdx.x; r < b.nrep; r += NT) {
        int np = vfl[r * FLAG_COUNT + FLAG_NPAIRS];
        if (reps[r].live && built(r)) np = vfl[r * FLAG_COUNT + FLAG_NEWPAIRS];
        np = min(np, reps[r].pcap);  // (above pcap only after an overflow)
        l.flags[r * FLAG_COUNT + FLAG_NPAIRS] = np;
        l.tile_start[r] = reps[r].live ? (np + b.tile - 1) / b.tile : 0;
    }
    __syncthreads();
    const int total = block_scan<NT>(l.tile_start, l.tile_start, b.nrep, part);
    if (threadIdx.x == 0) l.tile_start[b.nrep] = total;
}

// The end of a step's list build, by workgroup fb of nfb (64 threads each):
// the tile plan (the first of them) and the pair entries of every chunk of
// the replicas with FLAG_FILL, a quarter of a chunk per workgroup at a time; the cells
// are emptied for the next build.  part: 64 ints of LDS.
__device__ inline void fill_step(const BatchParams &b, const SysParams *reps, const ListPtrs &l, int fb, int nfb, int *part)
{
    if (l.gflags[G_FILL] == 0) return;
    if (fb == 0)
        plan<kChunk>(b, reps, l, part, [&](int r) { return reps[r].n > 0 && l.flags[r * FLAG_COUNT + FLAG_FILL] != 0; });
    // the replicas that rebuild, 64 at a time; their chunks dealt over
    // the fill workgroups from a replica-dependent start
    for (int r0 = 0; r0 < b.nrep; r0 += 64) {
        const int rl = r0 + (int)__lane_id();
        const bool bld = rl < b.nrep && reps[rl].live && reps[rl].n > 0 && l.flags[rl * FLAG_COUNT + FLAG_FILL] != 0;
        for (unsigned long long m = __ballot(bld); m != 0ull; m &= m - 1ull) {
            const int r = r0 + __builtin_ctzll(m);
            const SysParams &p = reps[r];
            const int c0 = p.off / kChunk, nc = (p.n + kChunk - 1) / kChunk;
            for (int k = (fb + nfb - (int)(((long long)r * 977) % nfb)) % nfb; k < nc * kFillParts; k += nfb)
                fill_part(b, p, l, c0 + k / kFillParts, k % kFillParts, false, true);
        }
    }
}

}  // namespace lb
}  // namespace dem

// Per-image cell lists, candidate lists and full neighbour lists.
//
// The neighbours of atom i are every (j, n) != (i, 0) with
//     r = (R_j - R_i) + ((n0 h_0 + n1 h_1) + n2 h_2),  (r_x r_x + r_y r_y) + r_z r_z < rc^2,
// evaluated in FP64 with every operation rounded on its own (no contraction), on the
// unwrapped positions R = R~ D.  This is the local environment of Sec. II.B, Eq. (4).
//
// Candidates (Verlet skin): a cell-list scan keeps every pair closer than
// rcl = rc + skin; each step re-tests the candidates with the exact inclusion test
// above, so the neighbour set is the one a full scan would give.  The candidates are
// rebuilt when a pair could have come from outside rcl: with h = h_ref (I + E) and
// d_i = |R_i - R_i,ref (I + E)|, a pair's separation at the build is at most
// (r + d_i + d_j) / (1 - |E|), so 2 max d_i + rcl |E| < skin keeps the list complete.
// R_ref is kept in FP32: each component within 2^-24 of its magnitude, so d_i measured
// against it is within 2^-24 |R_ref,i| (1 + |E|) of the true one, added to the bound.
//
// Kernels, in order (each a persistent walk over the items of every live band); bands of
// up to CFNEB_SKIN_IMAGE atoms take k_skin_image instead of all before k_cand, those of up
// to CFNEB_BIN_IMAGE k_skin_bins instead of k_skin_decide and the four bin kernels:
//   k_skin_check   (steps) the previous step's move of the atom rows; R = R~ D (and
//                  its fixed-point fractional coordinates); max_i d_i^2 per 1024-atom tile
//   k_skin_decide  max over an image's tiles, rebuild flag per image; a rebuild takes
//                  the current cell as reference
//   k_bin_assign   (rebuilds) wrapped fractional coordinate, bin id; the count atomic
//                  returns the atom's rank inside its bin
//   k_bin_scan     (rebuilds) exclusive prefix sum of the bin counts (one block per
//                  image, 4096 counts per pass, coalesced); zeroes the counts
//   k_bin_scatter  (rebuilds) atom -> bin-ordered 16-byte record (BinAtom)
//   k_bin_sort     (rebuilds) sort each bin by atom id, so lists are deterministic
//   k_cand         (rebuilds) pairs within rcl by groups of bins, a wave to a group (narrow
//                  cells, far images and crowded shares: two lanes to an atom); the packed
//                  candidate lists; R_ref = R
//   k_filter       (host readouts only: the force kernels test their candidates
//                  themselves) exact test of every candidate, packed entry-major
//                  neighbour lists (entry e of atom i at [e][i])
#include <type_traits>

#include "cfneb_dev.h"

namespace cfneb {

__device__ inline size_t bin_base(const BandDev& b, int slot) { return size_t(slot) * (b.nbcap + 1); }

// A lattice image (three counts) in 10-bit fields, as bin_assign stores it.
__device__ inline int img_n(int v, int k) { return ((v >> (10 * k)) & 0x3FF) - 512; }
// Three counts modulo 16 in the fields of a list entry.
__device__ inline uint32_t pack_images(int n0, int n1, int n2)
{
    return (uint32_t(n0 & 15) << 20) | (uint32_t(n1 & 15) << 24) | (uint32_t(n2 & 15) << 28);
}
__device__ inline const int* binfo_of(const BandDev& b, int slot, int field)
{
    return b.binfo + (size_t(slot) * 3 + field) * b.N;
}

// Fractional coordinates s = R h^-1 wrapped to [0, 1) and rounded to multiples of
// 2^-32 (1.0 wraps to 0); a non-finite coordinate gives 0 (the energy check reports
// the band).
__device__ inline uint4 fixed_fraction(const double* r, const double* hi)
{
    uint32_t u[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const double s = (r[0] * hi[q] + r[1] * hi[3 + q]) + r[2] * hi[6 + q];
        const double t = isfinite(s) ? s - floor(s) : 0.0;
        u[q] = uint32_t((unsigned long long)(long long)rint(t * 0x1p32));
    }
    return make_uint4(u[0], u[1], u[2], 0u);
}

// Four atoms i0, i0 + stride, ..: all loads are issued before any position is stored.  In
// a step, first the previous step's pending move of these atom rows (X += scale dt v',
// written back); R = R~ D (and its fixed-point fractional coordinates for FP32 LJ bands);
// m[0], m[1]: maximum of d_i^2 against the strained FP32 reference when a list exists
// (valid), and of |R_ref,i|^2 for its rounding.
struct SkinFrame {
    double D[9], E[9], hi[9];
    bool valid;
};
__device__ inline void skin_atoms(const BandDev& b, const cmem<BandState>* st, int slot, const SkinFrame& f, int i0,
                                  int stride, int all_images, double (&m)[2])
{
    constexpr int Q = CFNEB_TILE4 / CFNEB_TILE;
    gmem<uint32_t>* __restrict__ S = b.S ? gp(Ss(b, slot)) : nullptr;
    gmem<double>* __restrict__ X = gp(Xs(b, slot));
    const gmem<const float>* __restrict__ Rr = gp<const float>(b.Rref + size_t(slot) * slot_rows(b));
    double x[Q][3], a[Q][3];
    if (move_pending(st, all_images)) {  // uniform over the block
        // the previous step's move of these rows: X += scale (dt v')
        const gmem<const double>* __restrict__ V = gp<const double>(Vs(b, st->vcur, slot));
        const double sc = st->scale, dt = st->dt;
        double v[Q][3];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = i0 + q * stride;
            const bool in = i < b.N;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                x[q][c] = in ? X[size_t(c) * b.ld + i] : 0.0;
                v[q][c] = in ? V[size_t(c) * b.ld + i] : 0.0;
                a[q][c] = (in && f.valid) ? double(Rr[size_t(c) * b.ld + i]) : 0.0;
            }
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = i0 + q * stride;
            if (i >= b.N) continue;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                x[q][c] += sc * (dt * v[q][c]);
                X[size_t(c) * b.ld + i] = x[q][c];
            }
        }
    } else {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = i0 + q * stride;
            const bool in = i < b.N;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                x[q][c] = in ? X[size_t(c) * b.ld + i] : 0.0;
                a[q][c] = (in && f.valid) ? double(Rr[size_t(c) * b.ld + i]) : 0.0;
            }
        }
    }
    gmem<R3>* __restrict__ R = gp(Rs(b, slot));
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int i = i0 + q * stride;
        if (i >= b.N) continue;
        double r[3];
        for (int c = 0; c < 3; ++c) r[c] = (x[q][0] * f.D[c] + x[q][1] * f.D[3 + c]) + x[q][2] * f.D[6 + c];
        store3(R, i, r[0], r[1], r[2]);
        if (S) {
            const uint4 w = fixed_fraction(r, f.hi);
            S[3 * size_t(i)] = w.x;
            S[3 * size_t(i) + 1] = w.y;
            S[3 * size_t(i) + 2] = w.z;
        }
        if (f.valid) {
            double d2 = 0.0;
            for (int c = 0; c < 3; ++c) {
                const double ref = a[q][c] + ((a[q][0] * f.E[c] + a[q][1] * f.E[3 + c]) + a[q][2] * f.E[6 + c]);
                const double d = r[c] - ref;
                d2 += d * d;
            }
            m[0] = fmax(m[0], d2);
            m[1] = fmax(m[1], (a[q][0] * a[q][0] + a[q][1] * a[q][1]) + a[q][2] * a[q][2]);
        }
    }
}
__device__ inline SkinFrame skin_frame(const BandDev& b, int slot)
{
    const cmem<ImageGeom>* g = cp(b.geom + slot);
    SkinFrame f;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        f.D[q] = g->D[q];
        f.E[q] = g->E[q];
        f.hi[q] = g->hinv[q];
    }
    f.valid = cp(b.skst + slot)->valid != 0;
    return f;
}

// Large bands: 1024 atoms per item, four per thread; the tile's maxima go to its own slot
// (no atomics: many tiles per image would contend on one address).
__global__ void __launch_bounds__(CFNEB_TILE) k_skin_check(BatchDev bd, int all_images)
{
    __shared__ double lds[(CFNEB_TILE / 64) * 2];
    ItemLoopRO loop(bd, KIND_ATOM4, all_images);
    Item it;
    while (loop.next(it)) {
        const BandDev b = band_ro(bd, it.band);
        const cmem<BandState>* st = cp(b.st);
        if (band_stopped(st)) continue;  // uniform over the block
        const int slot = st->slot[it.image];
        const SkinFrame f = skin_frame(b, slot);
        double m[2] = {0.0, 0.0};
        skin_atoms(b, st, slot, f, it.tile * CFNEB_TILE4 + int(threadIdx.x), CFNEB_TILE, all_images, m);
        block_max<2>(m, lds);
        if (threadIdx.x == 0) {
            double* out = b.skmax + (size_t(slot) * kind_tiles(b, KIND_ATOM4) + it.tile) * 2;
            out[0] = m[0];
            out[1] = m[1];
        }
    }
}

// The decision for one image from its maxima; a rebuild takes the current cell as
// reference.  Returns whether the image rebuilds its candidates.
__device__ inline bool skin_decision(const BatchDev& bd, const BandDev& b, int slot, const double (&m)[2])
{
    SkinState& sk = b.skst[slot];
    const ImageGeom& g = b.geom[slot];
    bool rebuild = true;
    // the FP32 reference is within 2^-24 |R_ref,i| of the build positions, so every
    // displacement is within that times (1 + |E|) of the one measured against it
    const double dmax = sqrt(m[0]) + 0x1p-24 * (1.0 + 1e-6) * sqrt(m[1]) * (1.0 + g.enorm);
    if (b.skin > 0.0 && sk.valid) rebuild = !(2.0 * dmax + b.rcl * g.enorm < b.skin * (1.0 - 1e-6));
    sk.rebuild = rebuild ? 1 : 0;
    if (rebuild) {
        for (int q = 0; q < 9; ++q) {
            sk.href[q] = g.h[q];
            sk.hrefinv[q] = g.hinv[q];
        }
        sk.far = sk.uneven = 0;
        sk.valid = 1;
        *rebuild_flag(bd) = 1;
    }
    return rebuild;
}

// One block per band, sixteen threads per image: the maximum over the image's tile
// maxima (max is exact in any order), then the decision.
__global__ void __launch_bounds__(16 * CFNEB_MAX_IMAGES) k_skin_decide(BatchDev bd, int all_images)
{
    ItemLoop loop(bd, KIND_BAND, all_images);
    Item it;
    while (loop.next(it)) {
        const BandDev& b = bd.bands[it.band];
        if (!bins_by_tiles(b)) continue;
        const BandState* st = b.st;
        const int k = threadIdx.x >> 4, lane = threadIdx.x & 15;
        const bool act = !band_stopped(st) && k < b.Mcap && image_active(st, k, all_images);
        const int slot = act ? st->slot[k] : 0;
        const int nt = kind_tiles(b, KIND_ATOM4);
        double m[2] = {0.0, 0.0};
        if (act) {
            const gmem<const double>* mx = gp<const double>(b.skmax + size_t(slot) * nt * 2);
#pragma unroll 4
            for (int t = lane; t < nt; t += 16) {
                m[0] = fmax(m[0], mx[2 * t]);
                m[1] = fmax(m[1], mx[2 * t + 1]);
            }
        }
        for (int off = 8; off > 0; off >>= 1) {
            m[0] = fmax(m[0], __shfl_xor(m[0], off, 16));
            m[1] = fmax(m[1], __shfl_xor(m[1], off, 16));
        }
        if (act && lane == 0) skin_decision(bd, b, slot, m);
    }
}

// Bin of an atom and the lattice image it lies in, from its position.
__device__ inline int bin_of(const ImageGeom& g, const double4& ri, int (&img)[3])
{
    const double r[3] = {ri.x, ri.y, ri.z};
    int bi[3];
    for (int q = 0; q < 3; ++q) {
        const double s = (r[0] * g.hinv[q] + r[1] * g.hinv[3 + q]) + r[2] * g.hinv[6 + q];
        double fl = floor(s);
        if (!isfinite(fl) || fabs(fl) > 500.0) fl = 0.0;  // non-finite input: caught by the energy check
        img[q] = int(fl);
        const double sw = s - fl;
        int bq = int(floor(sw * g.nb[q]));
        bq = bq < 0 ? 0 : (bq >= g.nb[q] ? g.nb[q] - 1 : bq);
        bi[q] = bq;
    }
    return (bi[0] * g.nb[1] + bi[1]) * g.nb[2] + bi[2];
}
__device__ inline int pack_binfo_image(const int (&img)[3])
{
    return (img[0] + 512) | ((img[1] + 512) << 10) | ((img[2] + 512) << 20);
}
__device__ inline bool image_is_far(const int (&img)[3])
{
    return abs(img[0]) > 3 || abs(img[1]) > 3 || abs(img[2]) > 3;
}
// Atom i's record in bin order; its code carries the atom and 3 - im in each field, im its
// lattice image (within 3 of the cell: others take cand_item, which does not read it).
__device__ inline BinAtom bin_record(const ImageGeom& g, const double4& ri, int i, int im)
{
    const double n0 = img_n(im, 0), n1 = img_n(im, 1), n2 = img_n(im, 2);
    BinAtom a;
    a.x = float(ri.x - (n0 * g.h[0] + n1 * g.h[3] + n2 * g.h[6]));
    a.y = float(ri.y - (n0 * g.h[1] + n1 * g.h[4] + n2 * g.h[7]));
    a.z = float(ri.z - (n0 * g.h[2] + n1 * g.h[5] + n2 * g.h[8]));
    a.code = uint32_t(i) | pack_images(3 - img_n(im, 0), 3 - img_n(im, 1), 3 - img_n(im, 2));
    return a;
}

// Half-width bins go in runs of four: two are 17 % slower on 97,555 LJ atoms and 24 % on a
// request of 16,383, three 5 % faster and 7 % slower.  Full-width bins hold a quarter of the
// atoms (two or three), so their runs are longer: 12 bins from 16,385 atoms on, 8 below.
// Which is better goes by how a row's bins divide as much as by size (a row's bins are shared
// evenly among its groups); carbon, us a build with 8 | 12: diamond of 2,743 atoms x 11 images
// 44 | 49, 13,823 x 1 40 | 38, 13,823 x 22 99 | 101, 17,575 x 1 41 | 40, 46,655 x 1 50 | 40,
// 46,655 x 10 144 | 130, 63,999 x 7 133 | 138, 85,183 x 7 174 | 211, 97,335 x 5 147 | 133;
// graphite of 73,728 x 12 325 with 12, 390 with 4.
#define CAND_RUN 4
#define CAND_RUN_SPARSE 12
#define CAND_RUN_SMALL 8

// How the candidate scan shares out an image's bins: groups of up to `run` bins of a row along
// the third axis (gz to a row), `per` consecutive groups to each of its tiles.
struct CandShares {
    int gz, total, per;
};
template <typename G>
__device__ inline CandShares cand_shares(const G* g, int N)
{
    const int run = g->sub > 1 ? CAND_RUN : N > 16384 ? CAND_RUN_SPARSE : CAND_RUN_SMALL;
    const int tiles = (N + CFNEB_TILE_CAND - 1) / CFNEB_TILE_CAND;
    CandShares c;
    c.gz = (g->nb[2] + run - 1) / run;
    c.total = g->nb[0] * g->nb[1] * c.gz;
    c.per = (c.total + tiles - 1) / tiles;
    return c;
}
// Shares of more than three times the mean number of atoms (clusters, wires: most bins are
// empty and the others in a few rows) would hold a few waves while the rest of the chip waits;
// such images take the scan that shares out atoms (cand_item).  All threads of the block, the
// bins' starts in place.  A ball of 16,000 LJ atoms in twice its lattice's edge, one image, a
// step that builds its list: 945 us by groups, 223 us that way (463 before there were groups).
// The shares of a crystal reach 1.8 times the mean at most.
template <typename S>
__device__ inline void flag_uneven(const BandDev& b, const ImageGeom& g, int slot, const S* start)
{
    const CandShares c = cand_shares(&g, b.N);
    auto first_bin = [&](int q) {
        const int row = q / c.gz;
        return row * g.nb[2] + (q - row * c.gz) * g.nb[2] / c.gz;
    };
    for (int q = int(threadIdx.x) * c.per; q < c.total; q += int(blockDim.x) * c.per)
        if (int(start[first_bin(min(q + c.per, c.total))]) - int(start[first_bin(q)]) > 3 * CFNEB_TILE_CAND)
            b.skst[slot].uneven = 1;
}

// The bins of one image by one block of 1024 threads: counts, then starts, and the ids of
// each bin in LDS (16 bits each: at most CFNEB_BIN_IMAGE atoms).  Four atoms a thread at a
// time, so the loads of a round are in flight together.
__device__ void bins_of_image(const BandDev& b, const ImageGeom& g, int slot, unsigned short* start,
                              unsigned short* ids, int* wsum)
{
    constexpr int Q = 4;
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    const int N = b.N, nbins = g.nbins;
    unsigned* counts = reinterpret_cast<unsigned*>(start);  // two bins to a word
    for (int q = t; q <= nbins / 2; q += 1024) counts[q] = 0;
    __syncthreads();
    gmem<int>* __restrict__ info = gp(b.binfo + size_t(slot) * 3 * N);
    const gmem<const R3>* __restrict__ R = gp<const R3>(Rs(b, slot));
    for (int i0 = t; i0 < N; i0 += 1024 * Q) {
        double4 r[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) r[q] = load4(R, min(i0 + 1024 * q, N - 1));
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = i0 + 1024 * q;
            if (i >= N) break;
            int img[3];
            const int bin = bin_of(g, r[q], img), sh = (bin & 1) * 16;
            info[i] = bin;
            info[N + i] = int((atomicAdd(&counts[bin >> 1], 1u << sh) >> sh) & 0xFFFFu);
            info[2 * N + i] = pack_binfo_image(img);
            if (image_is_far(img)) b.skst[slot].far = 1;
        }
    }
    __syncthreads();
    // exclusive scan of the counts, a run of bins per thread
    const int per = (nbins + 1023) >> 10, q0 = min(t * per, nbins), q1 = min(q0 + per, nbins);
    int sum = 0;
    for (int q = q0; q < q1; ++q) sum += start[q];
    int incl = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(incl, off, 64);
        if (lane >= off) incl += y;
    }
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    int run = incl - sum;
    for (int w = 0; w < wid; ++w) run += wsum[w];
    gmem<int>* __restrict__ gstart = gp(b.bstart + bin_base(b, slot));
    for (int q = q0; q < q1; ++q) {
        const int c = start[q];
        start[q] = (unsigned short)run;
        gstart[q] = run;
        run += c;
    }
    if (t == 0) {
        start[nbins] = (unsigned short)N;
        gstart[nbins] = N;
    }
    __syncthreads();
    flag_uneven(b, g, slot, start);
    for (int i0 = t; i0 < N; i0 += 1024 * Q) {
        int bin[Q], rank[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = min(i0 + 1024 * q, N - 1);
            bin[q] = info[i];
            rank[q] = info[N + i];
        }
#pragma unroll
        for (int q = 0; q < Q; ++q)
            if (i0 + 1024 * q < N) ids[int(start[bin[q]]) + rank[q]] = (unsigned short)(i0 + 1024 * q);
    }
    __syncthreads();
    // an atom's place in its bin is the number of smaller ids there
    BinAtom* out = b.bpos + size_t(slot) * N;
    for (int i0 = t; i0 < N; i0 += 1024 * Q) {
        int bin[Q], im[Q];
        double4 r[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = min(i0 + 1024 * q, N - 1);
            bin[q] = info[i];
            im[q] = info[2 * N + i];
            r[q] = load4(R, i);
        }
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = i0 + 1024 * q;
            if (i >= N) break;
            const int lo = start[bin[q]], hi = start[bin[q] + 1];
            int pos = lo;
            for (int p = lo; p < hi; ++p) pos += int(ids[p]) < i ? 1 : 0;
            out[pos] = bin_record(g, r[q], i, im[q]);
        }
    }
    __syncthreads();
}

// Bands of up to CFNEB_SKIN_IMAGE atoms: one block per image takes the positions, the skin
// test, the decision and, on a rebuild, the bins, so the phases that are launches of their
// own for large bands (four of them idle on most steps) are block barriers here.
// Latency-bound.  Skin test and idle bin launches per step: 255 LJ atoms x 5 images 15 -> 7 us.
__global__ void __launch_bounds__(1024) k_skin_image(BatchDev bd, int all_images)
{
    __shared__ double lds[16 * 2];
    __shared__ alignas(4) unsigned short start[CFNEB_SKIN_IMAGE + 64 + 2];
    __shared__ unsigned short ids[CFNEB_SKIN_IMAGE];
    __shared__ int wsum[16];
    __shared__ int rebuild;
    const int t = threadIdx.x;
    ItemLoopRO loop(bd, KIND_SIMAGE, all_images);
    Item it;
    while (loop.next(it)) {
        const BandDev b = band_ro(bd, it.band);
        const cmem<BandState>* st = cp(b.st);
        if (band_stopped(st)) continue;  // uniform over the block
        const int slot = st->slot[it.image], N = b.N;
        double m[2] = {0.0, 0.0};
        {
            const SkinFrame f = skin_frame(b, slot);
            for (int i0 = t; i0 - t < N; i0 += 4096) skin_atoms(b, st, slot, f, i0, 1024, all_images, m);
        }
        block_max<2>(m, lds);
        if (t == 0) rebuild = skin_decision(bd, b, slot, m) ? 1 : 0;
        __syncthreads();
        if (!rebuild) continue;  // uniform (the next write of the flag is behind barriers)
        bins_of_image(b, b.geom[slot], slot, start, ids, wsum);
    }
}

// Bands of up to CFNEB_BIN_IMAGE atoms: one block per image takes the decision from the
// tiles' maxima (as k_skin_decide) and, on a rebuild, the bins.  Bound by launches when no
// image rebuilds, by one CU's round trips when one does (figures at CFNEB_BIN_IMAGE).
__global__ void __launch_bounds__(1024) k_skin_bins(BatchDev bd, int all_images)
{
    __shared__ alignas(4) unsigned short start[CFNEB_BIN_IMAGE + 64 + 2];
    __shared__ unsigned short ids[CFNEB_BIN_IMAGE];
    __shared__ int wsum[16];
    __shared__ int rebuild;
    ItemLoopRO loop(bd, KIND_BIMAGE, all_images);
    Item it;
    while (loop.next(it)) {
        const BandDev b = band_ro(bd, it.band);
        const cmem<BandState>* st = cp(b.st);
        if (band_stopped(st)) continue;  // uniform over the block
        const int slot = st->slot[it.image];
        if (threadIdx.x < 64) {
            const int nt = kind_tiles(b, KIND_ATOM4);
            const gmem<const double>* mx = gp<const double>(b.skmax + size_t(slot) * nt * 2);
            double m[2] = {0.0, 0.0};
            for (int k = threadIdx.x; k < nt; k += 64) {
                m[0] = fmax(m[0], mx[2 * k]);
                m[1] = fmax(m[1], mx[2 * k + 1]);
            }
            for (int off = 32; off > 0; off >>= 1) {
                m[0] = fmax(m[0], __shfl_xor(m[0], off, 64));
                m[1] = fmax(m[1], __shfl_xor(m[1], off, 64));
            }
            if (threadIdx.x == 0) rebuild = skin_decision(bd, b, slot, m) ? 1 : 0;
        }
        __syncthreads();
        if (rebuild) {  // uniform
            // a copy held in scalar registers (in k_skin_image it would cost the idle steps)
            const ImageGeom g = *(const ImageGeom*)cp(b.geom + slot);
            bins_of_image(b, g, slot, start, ids, wsum);
        }
        __syncthreads();
    }
}

__device__ void bin_assign_item(const BandDev& b, int slot, int i)
{
    int img[3];
    const int bin = bin_of(b.geom[slot], load4(gp<const R3>(Rs(b, slot)), i), img);
    const int rank = atomicAdd(&b.bcount[bin_base(b, slot) + bin], 1);
    int* info = b.binfo + size_t(slot) * 3 * b.N + i;
    info[0] = bin;
    info[b.N] = rank;
    info[2 * size_t(b.N)] = pack_binfo_image(img);
    if (image_is_far(img)) b.skst[slot].far = 1;
}

__global__ void __launch_bounds__(CFNEB_TILE) k_bin_assign(BatchDev bd, int all_images)
{
    if (*rebuild_flag(bd) == 0) return;  // no image rebuilds this step
    ItemLoop loop(bd, KIND_LATOM, all_images);
    Item it;
    while (loop.next(it)) {
        const BandDev& b = bd.bands[it.band];
        const BandState* st = b.st;
        const int i = it.tile * CFNEB_TILE + threadIdx.x;
        if (band_stopped(st) || i >= b.N) continue;
        const int slot = st->slot[it.image];
        if (!b.skst[slot].rebuild) continue;
        bin_assign_item(b, slot, i);
    }
}

// Exclusive scan of one image's counts, 4 per thread and 4096 per pass.
__device__ void bin_scan_item(const BandDev& b, int slot)
{
    __shared__ int wsum[16];
    __shared__ int carry_s;
    const int nbins = b.geom[slot].nbins;
    int* cnt = b.bcount + bin_base(b, slot);
    int* start = b.bstart + bin_base(b, slot);
    const int t = threadIdx.x, lane = t & 63, wid = t >> 6;
    int carry = 0;
    for (int base = 0; base < nbins; base += 4096) {
        const int idx = base + 4 * t;
        int c[4];
        for (int q = 0; q < 4; ++q) c[q] = (idx + q < nbins) ? cnt[idx + q] : 0;
        const int s1 = c[0] + c[1], s2 = s1 + c[2], tot = s2 + c[3];
        int incl = tot;
        for (int off = 1; off < 64; off <<= 1) {
            const int y = __shfl_up(incl, off, 64);
            if (lane >= off) incl += y;
        }
        if (lane == 63) wsum[wid] = incl;
        __syncthreads();
        if (t == 0) {
            int run = 0;
            for (int w = 0; w < 16; ++w) {
                const int v = wsum[w];
                wsum[w] = run;
                run += v;
            }
            carry_s = run;
        }
        __syncthreads();
        const int excl = carry + wsum[wid] + incl - tot;
        const int pre[4] = {0, c[0], s1, s2};
        for (int q = 0; q < 4; ++q)
            if (idx + q < nbins) {
                start[idx + q] = excl + pre[q];
                cnt[idx + q] = 0;
            }
        carry += carry_s;
        __syncthreads();
    }
    if (t == 0) start[nbins] = carry;
    __syncthreads();
    flag_uneven(b, b.geom[slot], slot, start);
}

__global__ void __launch_bounds__(1024) k_bin_scan(BatchDev bd, int all_images)
{
    if (*rebuild_flag(bd) == 0) return;  // no image rebuilds this step
    ItemLoop loop(bd, KIND_LIMAGE, all_images);
    Item it;
    while (loop.next(it)) {
        const BandDev& b = bd.bands[it.band];
        if (band_stopped(b.st)) continue;  // uniform over the block
        const int slot = b.st->slot[it.image];
        if (!b.skst[slot].rebuild) continue;  // uniform over the block
        bin_scan_item(b, slot);
    }
}

__global__ void __launch_bounds__(CFNEB_TILE) k_bin_scatter(BatchDev bd, int all_images)
{
    if (*rebuild_flag(bd) == 0) return;  // no image rebuilds this step
    ItemLoop loop(bd, KIND_LATOM, all_images);
    Item it;
    while (loop.next(it)) {
        const BandDev& b = bd.bands[it.band];
        const BandState* st = b.st;
        const int i = it.tile * CFNEB_TILE + threadIdx.x;
        if (band_stopped(st) || i >= b.N) continue;
        const int slot = st->slot[it.image];
        if (!b.skst[slot].rebuild) continue;
        const int pos = b.bstart[bin_base(b, slot) + binfo_of(b, slot, 0)[i]] + binfo_of(b, slot, 1)[i];
        const int im = binfo_of(b, slot, 2)[i];
        if (pos < 0 || pos >= b.N) continue;
        b.bpos[size_t(slot) * b.N + pos] = bin_record(b.geom[slot], load4(gp<const R3>(Rs(b, slot)), i), i, im);
    }
}

__global__ void __launch_bounds__(CFNEB_TILE) k_bin_sort(BatchDev bd, int all_images)
{
    if (*rebuild_flag(bd) == 0) return;  // no image rebuilds this step
    ItemLoop loop(bd, KIND_BIN, all_images);
    Item it;
    while (loop.next(it)) {
        const BandDev& b = bd.bands[it.band];
        const BandState* st = b.st;
        const int bin = it.tile * CFNEB_TILE + threadIdx.x;
        if (band_stopped(st)) continue;
        const int slot = st->slot[it.image];
        if (!b.skst[slot].rebuild || bin >= b.geom[slot].nbins) continue;
        const int* start = b.bstart + bin_base(b, slot);
        BinAtom* a = b.bpos + size_t(slot) * b.N;
        const int lo = start[bin], hi = min(start[bin + 1], b.N);
        for (int p = lo + 1; p < hi; ++p) {
            const BinAtom v = a[p];
            const int key = nbr_j(v.code);
            int q = p - 1;
            while (q >= lo && nbr_j(a[q].code) > key) {
                a[q + 1] = a[q];
                --q;
            }
            a[q + 1] = v;
        }
    }
}

__device__ inline void wrap_bin(int v, int nb, int& a, int& m)
{
    // periodic wrap without division (the stencil reach is small)
    a = v;
    m = 0;
    while (a < 0) {
        a += nb;
        --m;
    }
    while (a >= nb) {
        a -= nb;
        ++m;
    }
}

// Candidates of the atom of record p (bin order), two neighbouring lanes: every (j, n) within
// rcl in stencil order; R_ref = R.  Serves images whose stencil spans more than one neighbouring
// cell (cells narrower than rcl), with atoms more than three cells away, where 4-bit lattice
// images could wrap, or whose atoms crowd a share of the groups (flag_uneven).  Each lane takes
// four of eight records at a time.  FP32 between wrapped positions decides outside a band
// around rcl^2 (a component: 1 2^-24 of the largest coordinate L for the rounding of either
// position and for their difference, reach for that of the shift, 1 + reach for the sum), the
// exact FP64 test inside it; lattice images come with the records unless the image's atoms are
// far.
// Bound by the chain of a lane's record loads: 3 images of 55,295 LJ atoms written five cells
// away 255 us a build (570 us with one lane an atom and FP64 tests of gathered positions, one
// at a time), a step that builds 7 images of 102,399 atoms in a cell one lattice constant
// thick 1.05 ms (2.79 ms).
__device__ void cand_item(const BandDev& b, BandState* st, int slot, int p, int half)
{
    const cmem<ImageGeom>* g = cp(b.geom + slot);
    const gmem<const R3>* __restrict__ R = gp<const R3>(Rs(b, slot));
    const gmem<const int>* __restrict__ start = gp<const int>(b.bstart + bin_base(b, slot));
    const gmem<const float4>* __restrict__ bp =
        gp<const float4>(reinterpret_cast<const float4*>(b.bpos + size_t(slot) * b.N));
    const gmem<const int>* __restrict__ img = gp<const int>(binfo_of(b, slot, 2));
    const float4 me = load4(bp, p);
    const int i = nbr_j(__float_as_uint(me.w));
    const double4 r4 = load4(R, i);
    gmem<uint32_t>* __restrict__ cand = gp(Cs(b, slot));

    const double ri[3] = {r4.x, r4.y, r4.z};
    if (half == 0) {
        gmem<float>* __restrict__ Rr = gp(b.Rref + size_t(slot) * slot_rows(b));
        Rr[i] = float(ri[0]);
        Rr[b.ld + i] = float(ri[1]);
        Rr[2 * size_t(b.ld) + i] = float(ri[2]);
    }
    const int bin = binfo_of(b, slot, 0)[i], im = img[i];
    const int nb0 = g->nb[0], nb1 = g->nb[1], nb2 = g->nb[2];
    const int b0 = bin / (nb1 * nb2), b1 = (bin / nb2) % nb1, b2 = bin % nb2;
    const int r0 = g->reach[0], r1 = g->reach[1], r2 = g->reach[2];
    float big = 0.f;
    for (int c = 0; c < 3; ++c)
        big = fmaxf(big, float(fabs(g->h[c]) + fabs(g->h[3 + c]) + fabs(g->h[6 + c])) * 1.000001f);
    const float rcl = float(b.rcl), rclf2 = float(b.rcl2), u = 0x1p-24f;
    const float e = 1.7320509f * (4.f + 2.f * float(max(r0, max(r1, r2)))) * u * big;
    const float delta = 1.01f * (2.f * rcl * e + e * e) + 12.f * u * rclf2;
    const float lo2 = rclf2 - delta, hi2 = rclf2 + delta;
    const double rcl2 = b.rcl2;
    const int ccap = b.ccap, natoms = b.N;
    const bool far = cp(b.skst + slot)->far != 0;
    int cnt = 0;
    bool bad_shift = false;
    // records lo..hi-1 in bin order, seen from bin shift (m0, m1, m2)
    auto scan = [&](int lo, int hi, int m0, int m1, int m2) {
        const float sx = float(double(m0) * g->h[0] + double(m1) * g->h[3] + double(m2) * g->h[6]);
        const float sy = float(double(m0) * g->h[1] + double(m1) * g->h[4] + double(m2) * g->h[7]);
        const float sz = float(double(m0) * g->h[2] + double(m1) * g->h[5] + double(m2) * g->h[8]);
        constexpr int U = 4;
        for (int p0 = lo + U * half; p0 - U * half < hi; p0 += 2 * U) {
            float4 a[U];
            float rr[U];
            int j[U], imj[U];
            bool in[U];
#pragma unroll
            for (int w = 0; w < U; ++w) a[w] = load4(bp, min(p0 + w, hi - 1));
#pragma unroll
            for (int w = 0; w < U; ++w) {
                const float dx = (a[w].x - me.x) + sx, dy = (a[w].y - me.y) + sy, dz = (a[w].z - me.z) + sz;
                rr[w] = dx * dx + dy * dy + dz * dz;
                j[w] = nbr_j(__float_as_uint(a[w].w));
                const bool self = int(j[w] == i) & int((m0 | m1 | m2) == 0);
                in[w] = int(p0 + w < hi) & int(rr[w] < hi2) & int(!self);
            }
            if (far)  // uniform over the block; the record's own image fields wrap
#pragma unroll
                for (int w = 0; w < U; ++w) imj[w] = img[in[w] ? j[w] : i];
            uint32_t ent[U];
            int own = 0;
#pragma unroll
            for (int w = 0; w < U; ++w) {
                if (!in[w]) continue;
                int n[3] = {m0, m1, m2};
                for (int q = 0; q < 3; ++q)
                    n[q] += img_n(im, q) -
                            (far ? img_n(imj[w], q) : 3 - int((__float_as_uint(a[w].w) >> (20 + 4 * q)) & 15u));
                if (!(rr[w] < lo2)) {  // rare: FP32 cannot tell
                    const double4 rj = load4(R, j[w]);
                    double h[9], d[3];
                    for (int q = 0; q < 9; ++q) h[q] = g->h[q];
                    in[w] = exact_r2(ri, rj.x, rj.y, rj.z, h, n[0], n[1], n[2], d) < rcl2;
                }
                if (in[w] && (abs(n[0]) > CFNEB_MAX_SHIFT || abs(n[1]) > CFNEB_MAX_SHIFT || abs(n[2]) > CFNEB_MAX_SHIFT)) {
                    bad_shift = true;
                    in[w] = false;
                }
                ent[w] = pack_nbr(j[w], n[0], n[1], n[2]);
                own += in[w] ? 1 : 0;
            }
            const int other = dpp_i32<0xB1>(own);  // (the pair takes every branch together)
            int pos = cnt + (half ? other : 0);
            cnt += own + other;
#pragma unroll
            for (int w = 0; w < U; ++w) {
                if (!in[w]) continue;
                if (pos < ccap) cand[cand_at(ccap, i, pos)] = ent[w];
                ++pos;
            }
        }
    };
    // the bins b2 - r2 .. b2 + r2 of a row that lie in one cell are one run of records
    int unused, mlo, mhi;
    wrap_bin(b2 - r2, nb2, unused, mlo);
    wrap_bin(b2 + r2, nb2, unused, mhi);
    for (int dx = -r0; dx <= r0; ++dx) {
        int a0, m0;
        wrap_bin(b0 + dx, nb0, a0, m0);
        for (int dy = -r1; dy <= r1; ++dy) {
            int a1, m1;
            wrap_bin(b1 + dy, nb1, a1, m1);
            const int row = (a0 * nb1 + a1) * nb2;
            for (int m2 = mlo; m2 <= mhi; ++m2) {
                const int z0 = max(b2 - r2 - m2 * nb2, 0), z1 = min(b2 + r2 - m2 * nb2, nb2 - 1);
                scan(start[row + z0], min(start[row + z1 + 1], natoms), m0, m1, m2);
            }
        }
    }
    if (half == 0) b.ncand[size_t(slot) * b.N + i] = min(cnt, ccap);
    if (bad_shift) set_error(st, CFNEB_ECELL);
    if (cnt > ccap) set_error(st, CFNEB_ENEIGH);
}

// Every other image: one wave per group of up to CAND_RUN bins of a row along the third axis.
// The wave stages the records of the group's stencil in LDS once, shifted into the
// group's frame and cut to those within rcl of the group's bounding box; then, for each
// of the group's atoms in turn, 64 records are tested at a time, one per lane, and the
// lanes inside append their entries (ballot prefix).  A thread per atom instead walks its
// stencil as a serial chain of loads with every test and append diverging inside the wave.
// Bound by vector issue (62 % of the slots at 2.4 GHz on the lattice) and the scattered stores
// of the entries.  Building the lists of 24 images of 97,555 LJ atoms: 4,960 us with a thread
// per atom, 1,360 us this way (the perfect lattice 4,780 and 1,190).  Of the way there, in means
// over steps on which some images rebuild: lane sets held as scalar masks (a compare a test
// instead of three instructions) 489 -> 446 us, the record loop not unrolled (ten copies of it
// overran the instruction cache) 432, images added as fields that cannot carry 416.
//
// Distances are FP32 between wrapped positions: each component is within 10 2^-24 of the
// largest coordinate L (1 for the rounding of either position, 2 for the shift from the
// box's middle, at most 5 for sums no larger than the stencil; L is at least rcl here), so
// FP32 r^2 decides outside a band around rcl^2 and the exact FP64 test inside it: the
// list holds exactly the pairs that the FP64 test gives.
// (97,555 LJ atoms | request of 16,383: stages of 384 records 9 | 7 % slower; one atom to a
// record read 5 % slower, three or four 5 to 8 %.)
#define CAND_STAGE 512
#define CAND_SEGS 64
struct CandSeg {
    int lo, count;
    uint32_t images;
    float x, y, z;
};
struct CandLds {
    BinAtom rec[CAND_STAGE];
    CandSeg seg[CAND_SEGS];
};

__device__ inline float lane_f(float v, int t)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), t));
}
__device__ inline int lanes_below(unsigned long long mask)
{
    return __builtin_amdgcn_mbcnt_hi(unsigned(mask >> 32), __builtin_amdgcn_mbcnt_lo(unsigned(mask), 0u));
}
// The lanes of the (whole) wave where a condition holds, and the condition of a lane set:
// scalar registers both ways.
__device__ inline unsigned long long lanes_where(bool c) { return __builtin_amdgcn_ballot_w64(c); }
__device__ inline bool in_lanes(unsigned long long m) { return __builtin_amdgcn_inverse_ballot_w64(m); }
// Minimum over the whole wave, in every lane.
__device__ inline float wave_fmin(float v)
{
    v = fminf(v, __int_as_float(dpp_i32<0xB1>(__float_as_int(v))));
    v = fminf(v, __int_as_float(dpp_i32<0x4E>(__float_as_int(v))));
    v = fminf(v, __int_as_float(dpp_i32<0x141>(__float_as_int(v))));
    v = fminf(v, __int_as_float(dpp_i32<0x140>(__float_as_int(v))));
    const auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fminf(__uint_as_float(s[0]), __uint_as_float(s[1]));
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fminf(__uint_as_float(t[0]), __uint_as_float(t[1]));
}
// A record by its byte offset from a uniform base (fewer than 2^20 records).
__device__ inline const gmem<const float4>* at_byte(const gmem<const float4>* p, uint32_t off)
{
    return reinterpret_cast<const gmem<const float4>*>(reinterpret_cast<const gmem<const char>*>(p) + off);
}
// LDS written by some lanes of a wave and read by others of the same wave.
__device__ inline void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ inline bool cand_by_groups(const cmem<ImageGeom>* g, const cmem<SkinState>* sk)
{
    const int r = g->sub;
    return int((sk->far | sk->uneven) == 0) & int(g->reach[0] == r) & int(g->reach[1] == r) & int(g->reach[2] == r) &
           int(g->nb[0] >= r) & int(g->nb[1] >= r) & int(g->nb[2] >= r);
}

__device__ void cand_group(const BandDev& b, BandState* st, const cmem<ImageGeom>* g, int slot, int q, int gz,
                           CandLds& lds)
{
    const int lane = int(threadIdx.x) & 63;
    const int nb0 = g->nb[0], nb1 = g->nb[1], nb2 = g->nb[2], r = g->sub, N = b.N, ccap = b.ccap;
    const int row = q / gz, zg = q - row * gz, z0 = zg * nb2 / gz, z1 = (zg + 1) * nb2 / gz;
    const int b0 = row / nb1, b1 = row - b0 * nb1;
    const gmem<const int>* __restrict__ start = gp<const int>(b.bstart + bin_base(b, slot));
    const int first = uni(start[row * nb2 + z0]), last = uni(min(start[row * nb2 + z1], N));
    if (first >= last) return;  // uniform over the wave
    const gmem<const float4>* __restrict__ bp =
        gp<const float4>(reinterpret_cast<const float4*>(b.bpos + size_t(slot) * N));
    const gmem<const R3>* __restrict__ R = gp<const R3>(Rs(b, slot));
    float big = 0.f;
    for (int c = 0; c < 3; ++c)
        big = fmaxf(big, float(fabs(g->h[c]) + fabs(g->h[3 + c]) + fabs(g->h[6 + c])) * 1.000001f);
    const float rcl = float(b.rcl), rcl2 = float(b.rcl2), u = 0x1p-24f;
    const float e = 1.7320509f * 10.f * u * big;
    const float delta = 1.01f * (2.f * rcl * e + e * e) + 12.f * u * rcl2;
    const float lo2 = uni(rcl2 - delta), hi2 = uni(rcl2 + delta);
    const int width = 2 * r + 1, zlo = z0 - r, zhi = z1 - 1 + r;
    const int mlo = zlo < 0 ? -1 : 0, nseg = (zhi >= nb2 ? 1 : 0) - mlo + 1;
    const int segs = width * width * nseg;
    for (int a0 = first; a0 < last; a0 += 64) {
        // lane l holds atom l of the group
        const int na = min(64, last - a0);
        const float4 me = load4(bp, a0 + min(lane, na - 1));
        const uint32_t mec = __float_as_uint(me.w);
        const int id = nbr_j(mec);
        // an entry's fields are m + im_i - im_j + 8, in [1, 15]: sums of fields that never
        // carry, im_i + 3 here, m + 2 of the stencil's cell, 3 - im_j of the record
        const uint32_t mine = 0x66600000u - (mec & 0xFFF00000u);
        int cnt = 0;  // of lane's atom
        // atoms of one lattice image at a time (nearly always all of them), so the staged
        // records carry finished entries
        unsigned long long todo = na == 64 ? ~0ull : (1ull << na) - 1ull;
        while (todo) {
            const uint32_t image = uint32_t(__builtin_amdgcn_readlane(int(mine), __ffsll(todo) - 1));
            const bool part = mine == image && lane < na;
            const unsigned long long members = __ballot(part);
            todo &= ~members;
            float bx0 = part ? me.x : 1e30f, bx1 = part ? me.x : -1e30f, by0 = part ? me.y : 1e30f;
            float by1 = part ? me.y : -1e30f, bz0 = part ? me.z : 1e30f, bz1 = part ? me.z : -1e30f;
            bx0 = wave_fmin(bx0), by0 = wave_fmin(by0), bz0 = wave_fmin(bz0);
            bx1 = -wave_fmin(-bx1), by1 = -wave_fmin(-by1), bz1 = -wave_fmin(-bz1);
            // positions from here on are relative to the box's middle
            const float mx = 0.5f * (bx0 + bx1), my = 0.5f * (by0 + by1), mz = 0.5f * (bz0 + bz1);
            const float px = me.x - mx, py = me.y - my, pz = me.z - mz;
            const float wx = fmaxf(bx1 - mx, mx - bx0), wy = fmaxf(by1 - my, my - by0), wz = fmaxf(bz1 - mz, mz - bz0);
            int n = 0;  // staged records
            // every member against the staged records, two atoms to a record read
            auto test = [&]() {
                const int full = uni((n + 63) & ~63);
                if (n + lane < full) lds.rec[n + lane].x = 3e18f;  // outside of any cutoff
                wave_lds_fence();
                constexpr int V = 2;
                for (unsigned long long left = members; left;) {
                    float xi[V], yi[V], zi[V], hi[V];
                    uint32_t self[V];
                    int t[V], i[V], k[V];
                    uint32_t* out[V];
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        hi[v] = left ? hi2 : -1.f;  // an odd last atom has no partner
                        t[v] = left ? __ffsll(left) - 1 : t[0];
                        left &= left - 1;
                        xi[v] = lane_f(px, t[v]);
                        yi[v] = lane_f(py, t[v]);
                        zi[v] = lane_f(pz, t[v]);
                        i[v] = __builtin_amdgcn_readlane(id, t[v]);
                        k[v] = __builtin_amdgcn_readlane(cnt, t[v]);
                        self[v] = uint32_t(i[v]) | 0x88800000u;
                        out[v] = uni(Cs(b, slot) + cand_at(ccap, i[v], 0));
                    }
                    float4 next = *reinterpret_cast<const float4*>(&lds.rec[lane]);
#pragma unroll 1
                    for (int c = 0; c < full; c += 64) {
                        const float4 rec = next;
                        next = *reinterpret_cast<const float4*>(&lds.rec[min(c + 64, CAND_STAGE - 64) + lane]);
                        const uint32_t ent = __float_as_uint(rec.w);
                        // lane sets as scalar masks: the tests cost a compare each
                        float r2[V];
                        unsigned long long in[V], near[V], some = 0;
#pragma unroll
                        for (int v = 0; v < V; ++v) {
                            const float dx = rec.x - xi[v], dy = rec.y - yi[v], dz = rec.z - zi[v];
                            r2[v] = dx * dx + dy * dy + dz * dz;
                            in[v] = lanes_where(r2[v] < hi[v]) & lanes_where(ent != self[v]);
                            near[v] = in[v] & lanes_where(r2[v] >= lo2);
                            some |= near[v];
                        }
                        if (some) {  // rare: FP32 cannot tell
                            for (int v = 0; v < V; ++v) {
                                bool out_of = false;
                                if (in_lanes(near[v])) {
                                    const double4 p = load4(R, i[v]), o = load4(R, nbr_j(ent));
                                    const double ri[3] = {p.x, p.y, p.z};
                                    double h[9], d[3];
                                    for (int w = 0; w < 9; ++w) h[w] = g->h[w];
                                    const double rr = exact_r2(ri, o.x, o.y, o.z, h, nbr_n(ent, 0), nbr_n(ent, 1),
                                                               nbr_n(ent, 2), d);
                                    out_of = !(rr < b.rcl2);
                                }
                                in[v] &= ~lanes_where(out_of);
                            }
                        }
#pragma unroll
                        for (int v = 0; v < V; ++v) {
                            const int pos = k[v] + lanes_below(in[v]);
                            k[v] += int(__popcll(in[v]));
                            if (k[v] > ccap) in[v] &= lanes_where(pos < ccap);  // uniform
                            // entry pos at word (pos / 4) 256 + pos % 4 of the atom's column
                            const uint32_t off = (uint32_t(pos) << 8) - __umul24(uint32_t(pos) & 3u, 252u);
                            gmem<char>* at = gp(reinterpret_cast<char*>(out[v])) + off;
                            if (in_lanes(in[v])) *reinterpret_cast<gmem<uint32_t>*>(at) = ent;
                        }
                    }
#pragma unroll
                    for (int v = V - 1; v >= 0; --v) cnt = lane == t[v] ? k[v] : cnt;
                }
                wave_lds_fence();
                n = 0;
            };
            for (int s0 = 0; s0 < segs; s0 += CAND_SEGS) {
                // lane l: the run of records of segment s0 + l (a stencil row within one cell)
                const int s = s0 + lane, ns = min(CAND_SEGS, segs - s0);
                if (lane < ns) {
                    const int rr = s / nseg, m2 = mlo + s - rr * nseg;
                    const int dx = rr / width - r, dy = rr - (rr / width) * width - r;
                    int c0, m0, c1, m1;
                    wrap_bin(b0 + dx, nb0, c0, m0);
                    wrap_bin(b1 + dy, nb1, c1, m1);
                    const int base = (c0 * nb1 + c1) * nb2;
                    const int zs = max(zlo - m2 * nb2, 0), ze = min(zhi - m2 * nb2, nb2 - 1) + 1;
                    CandSeg sg;
                    sg.lo = start[base + zs];
                    sg.count = min(start[base + ze], N) - sg.lo;
                    sg.images = pack_images(m0 + 2, m1 + 2, m2 + 2) + image;
                    sg.x = float(double(m0) * g->h[0] + double(m1) * g->h[3] + double(m2) * g->h[6] - double(mx));
                    sg.y = float(double(m0) * g->h[1] + double(m1) * g->h[4] + double(m2) * g->h[7] - double(my));
                    sg.z = float(double(m0) * g->h[2] + double(m1) * g->h[5] + double(m2) * g->h[8] - double(mz));
                    lds.seg[lane] = sg;
                }
                wave_lds_fence();
                // 32 lanes to a segment; the loads of ten segments are in flight together, so
                // a 3 x 3 stencil takes one round and a 5 x 5 three (a longer segment, of a
                // clustered structure, takes further rounds): 412 us with eight, 399 with ten
                constexpr int U = 5;
                for (int p = 0; p < ns; p += 2 * U) {
                    for (int k0 = 0;; k0 += 32) {
                        float4 a[U];
                        CandSeg sg[U];
                        const int k = k0 + (lane & 31);
                        int more = 0;
#pragma unroll
                        for (int w = 0; w < U; ++w) {
                            const int sw = p + 2 * w + (lane >> 5);
                            sg[w] = lds.seg[min(sw, ns - 1)];
                            if (sw >= ns) sg[w].count = 0;
                            more |= int(k0 + 32 < sg[w].count);
                            a[w] = load4(at_byte(bp, uint32_t(k < sg[w].count ? sg[w].lo + k : first) * 16u), 0);
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int w = 0; w < U; ++w) {
                            if (n + 64 > CAND_STAGE) test();
                            a[w].x += sg[w].x;
                            a[w].y += sg[w].y;
                            a[w].z += sg[w].z;
                            const float ex = fmaxf(fabsf(a[w].x) - wx, 0.f);
                            const float ey = fmaxf(fabsf(a[w].y) - wy, 0.f);
                            const float ez = fmaxf(fabsf(a[w].z) - wz, 0.f);
                            const bool keep = int(k < sg[w].count) & int(ex * ex + ey * ey + ez * ez < hi2);
                            const unsigned long long mask = __ballot(keep);
                            if (keep) {
                                a[w].w = __uint_as_float(__float_as_uint(a[w].w) + sg[w].images);
                                *reinterpret_cast<float4*>(&lds.rec[n + lanes_below(mask)]) = a[w];
                            }
                            n = uni(n + int(__popcll(mask)));
                        }
                        if (!__any(more)) break;
                    }
                }
                wave_lds_fence();
            }
            test();
        }
        if (lane < na) {
            b.ncand[size_t(slot) * N + id] = min(cnt, ccap);
            if (cnt > ccap) set_error(st, CFNEB_ENEIGH);
            const double4 r4 = load4(R, id);
            gmem<float>* __restrict__ Rr = gp(b.Rref + size_t(slot) * slot_rows(b));
            Rr[id] = float(r4.x);
            Rr[b.ld + id] = float(r4.y);
            Rr[2 * size_t(b.ld) + id] = float(r4.z);
        }
    }
}

__global__ void __launch_bounds__(CFNEB_TILE) __attribute__((amdgpu_waves_per_eu(4)))
k_cand(BatchDev bd, int all_images)
{
    __shared__ CandLds lds[CFNEB_WAVES];
    if (*rebuild_flag(bd) == 0) return;  // no image rebuilds this step
    Item it;
    int others = 0;
    ItemLoopRO loop(bd, KIND_CAND, all_images);
    while (loop.next(it)) {
        const BandDev b = band_ro(bd, it.band);
        const cmem<BandState>* st = cp(b.st);
        if (band_stopped(st)) continue;
        const int slot = st->slot[it.image];
        const cmem<SkinState>* sk = cp(b.skst + slot);
        if (!sk->rebuild) continue;
        const cmem<ImageGeom>* g = cp(b.geom + slot);
        if (!cand_by_groups(g, sk)) {
            others = 1;
            continue;
        }
        // the tiles of an image share its groups evenly, in runs
        const CandShares c = cand_shares(g, b.N);
        const int end = min((it.tile + 1) * c.per, c.total), wave = uni(int(threadIdx.x) >> 6);
        // (the waves take turns at the first group, so an uneven share goes round)
        const int turn = (wave + it.tile) & (CFNEB_WAVES - 1);
        for (int q = it.tile * c.per + turn; q < end; q += CFNEB_WAVES) cand_group(b, b.st, g, slot, q, c.gz, lds[wave]);
    }
    // the images that groups do not serve, in a walk of their own: inside the one above their
    // code costs it scalar registers (two LJ bands, no image taking it: 113.6 -> 115.6 us)
    if (uni(others) == 0) return;  // uniform over the wave (no barrier follows)
    ItemLoopRO again(bd, KIND_CAND, all_images);
    while (again.next(it)) {
        const BandDev b = band_ro(bd, it.band);
        const cmem<BandState>* st = cp(b.st);
        if (band_stopped(st)) continue;
        const int slot = st->slot[it.image];
        const cmem<SkinState>* sk = cp(b.skst + slot);
        if (!sk->rebuild || cand_by_groups(cp(b.geom + slot), sk)) continue;
        const int p = it.tile * CFNEB_TILE_CAND + (int(threadIdx.x) >> 1);
        if (p < b.N) cand_item(b, b.st, slot, p, int(threadIdx.x) & 1);
    }
}

// Exact test of atom i's candidates with the current R and h: the packed neighbour
// list.  Four candidates at a time: one load of their entries, then their positions in
// flight together before any test (entries past the last candidate are in-bounds atoms;
// the tests stop there).
__device__ void filter_item(const BandDev& b, BandState* st, int slot, int i)
{
    const ImageGeom& g = b.geom[slot];
    const gmem<const R3>* __restrict__ R = gp<const R3>(Rs(b, slot));
    const size_t N = b.N;
    const gmem<const uint4>* __restrict__ cand = gp<const uint4>(reinterpret_cast<const uint4*>(Cs(b, slot)));
    gmem<uint32_t>* __restrict__ nbr = gp(b.nbr + size_t(slot) * b.cap * N);
    double h[9];
    for (int q = 0; q < 9; ++q) h[q] = g.h[q];
    const double4 r4 = load4(R, i);
    const double ri[3] = {r4.x, r4.y, r4.z};
    const int nc = gp<const int>(b.ncand)[size_t(slot) * N + i];
    const double rc2 = b.rc2;
    const int cap = b.cap;
    int cnt = 0;
    constexpr int U = 4;
    for (int e0 = 0; e0 < nc; e0 += U) {
        const uint4 e4 = load4(cand, cand_at(b.ccap, i, e0) >> 2);
        const uint32_t ent[U] = {e4.x, e4.y, e4.z, e4.w};
        double4 rj[U];
#pragma unroll
        for (int u = 0; u < U; ++u) rj[u] = load4(R, nbr_j(ent[u]));
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (e0 + u >= nc) break;
            double d[3];
            const double rr = exact_r2(ri, rj[u].x, rj[u].y, rj[u].z, h, nbr_n(ent[u], 0), nbr_n(ent[u], 1),
                                       nbr_n(ent[u], 2), d);
            if (!(rr < rc2)) continue;
            if (cnt < cap) nbr[size_t(cnt) * N + i] = ent[u];
            ++cnt;
        }
    }
    gp(b.ncnt)[size_t(slot) * N + i] = cnt;
    if (cnt > cap) set_error(st, CFNEB_ENEIGH);
}

// vmask: the band variants (potential, force precision) this launch serves
__global__ void __launch_bounds__(CFNEB_TILE) k_filter(BatchDev bd, int all_images, unsigned vmask, int ignore_stop)
{
    ItemLoop loop(bd, KIND_ATOM, all_images);
    Item it;
    while (loop.next(it)) {
        const BandDev& b = bd.bands[it.band];
        if (!((vmask >> band_variant(b)) & 1u)) continue;
        BandState* st = b.st;
        const int i = it.tile * CFNEB_TILE + threadIdx.x;
        if ((!ignore_stop && band_stopped(st)) || i >= b.N) continue;
        filter_item(b, st, st->slot[it.image], i);
    }
}

__global__ void k_skin_hold(BatchDev bd, int hold)
{
    for (int q = int(blockIdx.x); q < bd.cap; q += int(gridDim.x)) {
        if (!bd.live[q]) continue;
        const BandDev& b = bd.bands[q];
        for (int slot = int(threadIdx.x); slot < b.Mcap; slot += int(blockDim.x)) {
            SkinState& sk = b.skst[slot];
            if (hold) {
                sk.held = sk.rebuild;
                sk.rebuild = 0;
            } else {
                sk.rebuild = sk.held;
            }
        }
    }
}

void launch_skin_hold(const Launch& L, int hold, hipStream_t s)
{
    k_skin_hold<<<L.g[KIND_BAND], 64, 0, s>>>(L.bd, hold);
}

void launch_skin(const Launch& L, int all_images, hipStream_t s)
{
    if (L.variants & (1u << VARIANT_SKIN_IMAGE)) k_skin_image<<<L.g[KIND_SIMAGE], 1024, 0, s>>>(L.bd, all_images);
    if (!(L.variants & (1u << VARIANT_BIN_IMAGE | 1u << VARIANT_BIN_TILES))) return;
    k_skin_check<<<L.g[KIND_ATOM4], CFNEB_TILE, 0, s>>>(L.bd, all_images);
    if (L.variants & (1u << VARIANT_BIN_IMAGE)) k_skin_bins<<<L.g[KIND_BIMAGE], 1024, 0, s>>>(L.bd, all_images);
    if (!(L.variants & (1u << VARIANT_BIN_TILES))) return;
    k_skin_decide<<<L.g[KIND_BAND], 16 * CFNEB_MAX_IMAGES, 0, s>>>(L.bd, all_images);
}

void launch_bins(const Launch& L, int all_images, hipStream_t s)
{
    if (!(L.variants & (1u << VARIANT_BIN_TILES))) return;
    k_bin_assign<<<L.g[KIND_LATOM], CFNEB_TILE, 0, s>>>(L.bd, all_images);
    k_bin_scan<<<L.g[KIND_LIMAGE], 1024, 0, s>>>(L.bd, all_images);
    k_bin_scatter<<<L.g[KIND_LATOM], CFNEB_TILE, 0, s>>>(L.bd, all_images);
    k_bin_sort<<<L.g[KIND_BIN], CFNEB_TILE, 0, s>>>(L.bd, all_images);
}

void launch_list(const Launch& L, int all_images, hipStream_t s)
{
    k_cand<<<L.g[KIND_CAND], CFNEB_TILE, 0, s>>>(L.bd, all_images);
}

// The force kernels of both potentials test their candidates themselves; a step
// writes no packed neighbour list.
void launch_filter(const Launch& L, int all_images, hipStream_t s)
{
    (void)L;
    (void)all_images;
    (void)s;
}

// Packed neighbour lists of every image of the table, for a host readout (the step
// path keeps candidates only): the exact test of the current candidates on the
// positions and cell of the last evaluation.
void launch_neighbour_lists(const Launch& L, hipStream_t s)
{
    launch_plan(L, 1, 1, s);
    k_filter<<<L.g[KIND_ATOM], CFNEB_TILE, 0, s>>>(L.bd, 1, (1u << NVARIANT) - 1u, 1);
}

}  // namespace cfneb

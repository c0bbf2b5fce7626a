// Voronoi ("lattice-free") cell list on gfx950: the online k-means update of the
// Spatial Searching Algorithm section, batched over every system of a context.
//
//   E-step   exact nearest centroid per particle (FP64 distance of the
//            neighbour-set definition, ties to the lower index), warm-started
//            from the particle's current cell -- the paper's warm-start
//            heuristic -- and certified by an expanding search over a uniform
//            grid of centroids (the GPU stand-in for its k-d tree).
//   M-step   the particles counted and ordered by owning cell (stable in their
//            order before), and each centroid moved to the mean of its lipid
//            members.
//   Morton   centroids ordered along a Morton curve (21 bits per axis), cells
//            renumbered, and the particles moved to their cells' new places:
//            the two-level reordering.
//   lists    cell radii, the cell-pair list (sphere test with skin) and
//            per-particle neighbour lists in 64-particle ELL chunks.
//
// Every kernel is predicated on SysScal::rebuild so that one launch serves all
// systems that update at this step; the others are untouched.
#include "rbc_dev.h"

#include <climits>
#include <type_traits>

namespace rbc {

// ------------------------------------------------------------------ helpers

// A running maximum that many waves raise: the atomic is issued only when the value
// read (never above the true running maximum) is smaller, so that most waves skip the
// serialised same-address atomic.
template <class T>
__device__ __forceinline__ void max_if_larger(T *p, T v) {
    if (v > __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(p, v);
}

// Wavefront scans by DPP lane moves (row shifts 1, 2, 4, 8, then each row's last lane into
// the next rows): seven register instructions, where a shuffle through LDS takes about 130
// cycles for each of six steps.
template <int CTRL, int ROWS>
__device__ __forceinline__ int dpp_or0(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ int wave_incl_scan(int v) {
    v += dpp_or0<0x111, 0xf>(v);
    v += dpp_or0<0x112, 0xf>(v);
    v += dpp_or0<0x114, 0xf>(v);
    v += dpp_or0<0x118, 0xf>(v);
    v += dpp_or0<0x142, 0xa>(v);
    v += dpp_or0<0x143, 0xc>(v);
    return v;
}

// The largest of 64 non-negative values, on every lane.
__device__ __forceinline__ int wave_max_int(int v) {
    v = max(v, dpp_or0<0x111, 0xf>(v));
    v = max(v, dpp_or0<0x112, 0xf>(v));
    v = max(v, dpp_or0<0x114, 0xf>(v));
    v = max(v, dpp_or0<0x118, 0xf>(v));
    v = max(v, dpp_or0<0x142, 0xa>(v));
    v = max(v, dpp_or0<0x143, 0xc>(v));
    return __builtin_amdgcn_readlane(v, WAVE - 1);
}

// Smallest and largest of 64 values by the same lane moves, in the last lane (of 16 in each
// row's last lane with four steps).
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or(double old, double v) {
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(old), __double2loint(v), CTRL, ROWS, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(old), __double2hiint(v), CTRL, ROWS, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row_max(double v) {
    v = fmax(v, dpp_or<0x111, 0xf>(-INFINITY, v));
    v = fmax(v, dpp_or<0x112, 0xf>(-INFINITY, v));
    v = fmax(v, dpp_or<0x114, 0xf>(-INFINITY, v));
    return fmax(v, dpp_or<0x118, 0xf>(-INFINITY, v));
}
__device__ __forceinline__ double row_min(double v) {
    v = fmin(v, dpp_or<0x111, 0xf>(INFINITY, v));
    v = fmin(v, dpp_or<0x112, 0xf>(INFINITY, v));
    v = fmin(v, dpp_or<0x114, 0xf>(INFINITY, v));
    return fmin(v, dpp_or<0x118, 0xf>(INFINITY, v));
}
__device__ __forceinline__ double wave_max(double v) {
    v = row_max(v);
    v = fmax(v, dpp_or<0x142, 0xa>(-INFINITY, v));
    return fmax(v, dpp_or<0x143, 0xc>(-INFINITY, v));
}
__device__ __forceinline__ double wave_min(double v) {
    v = row_min(v);
    v = fmin(v, dpp_or<0x142, 0xa>(INFINITY, v));
    return fmin(v, dpp_or<0x143, 0xc>(INFINITY, v));
}

// Exclusive scan across the block (blockDim.x a multiple of 64, <= 1024).
__device__ int block_excl_scan(int v, int *s_w, int &total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int x = wave_incl_scan(v);
    if (lane == 63) s_w[w] = x;
    __syncthreads();
    int base = 0;
    total = 0;
    for (int q = 0; q < nw; ++q) {
        if (q < w) base += s_w[q];
        total += s_w[q];
    }
    __syncthreads();
    return base + x - v;
}

// In-place exclusive scan of a[0..n) by one block; a[n] receives the total.
__device__ void block_scan_array(int *a, int n, int *s_w) {
    int carry = 0;
    const int per = 4;
    for (int base = 0; base < n; base += blockDim.x * per) {
        int v[per];
        int loc = 0;
        for (int q = 0; q < per; ++q) {
            int idx = base + threadIdx.x * per + q;
            v[q] = (idx < n) ? a[idx] : 0;
            loc += v[q];
        }
        int tot;
        int ex = block_excl_scan(loc, s_w, tot);
        int run = carry + ex;
        for (int q = 0; q < per; ++q) {
            int idx = base + threadIdx.x * per + q;
            if (idx < n) a[idx] = run;
            run += v[q];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) a[n] = carry;
    __syncthreads();
}

#define SYS_FROM(map) \
    const int s = find_sys(L_maps.map, L_maps.nsys, blockIdx.x); \
    const SysDev &S = Sd[s]; \
    const int lb = blockIdx.x - L_maps.map[s];

// ------------------------------------------------------------------ rebuild flags

// The rebuild flags of every system from the mask, and the block maps restricted to the
// systems that rebuild (the others get no blocks), so that an update launches only the
// rebuilding systems' blocks.  The block counts per system match the full maps built on
// the host; one block of MAX_SLOTS threads.
__global__ __launch_bounds__(MAX_SLOTS) void k_set_rebuild(const SysDev *Sd, int nsys, unsigned long long m0,
                                                           unsigned long long m1, unsigned long long m2,
                                                           unsigned long long m3, int32_t *out) {
    __shared__ int s_w[16];
    const int s = threadIdx.x;
    int cnt[5] = {0, 0, 0, 0, 0};
    if (s < nsys) {
        const unsigned long long w = (s < 64) ? m0 : (s < 128) ? m1 : (s < 192) ? m2 : m3;
        const int bit = (int)((w >> (s & 63)) & 1ull);
        const SysDev &S = Sd[s];
        SysScal *sc = S.sc;
        sc->rebuild = bit;
        if (bit) {
            sc->rmax = 0ull;
            sc->nlrows = 0;
            sc->cnbr_maxrow = 0;
            sc->level = 0;
            sc->err &= ~(ERR_NLIST | ERR_NPAIRS | ERR_CNBR | ERR_ASSIGN);
            if (S.n > 0) {
                cnt[0] = (S.n + BLOCK - 1) / BLOCK;
                cnt[1] = (S.k + BLOCK - 1) / BLOCK;
                cnt[2] = S.ntile_s;
                cnt[3] = (S.k + SCAN_TILE - 1) / SCAN_TILE;
                cnt[4] = (S.gcap + SCAN_TILE - 1) / SCAN_TILE;
            }
        }
    }
    for (int m = 0; m < 5; ++m) {
        int tot;
        const int ex = block_excl_scan(cnt[m], s_w, tot);
        if (s <= nsys) out[m * (nsys + 1) + s] = ex;     // entry nsys receives the total
        if (s == 0 && nsys == MAX_SLOTS) out[m * (nsys + 1) + nsys] = tot;
    }
}

// ------------------------------------------------------------------ packing

__device__ void pack_one(const SysDev &S, const double *x, const double *n, const int32_t *type, const double *v,
                       const double *w) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= S.n) return;
    const int t = type[i];
    D4 p = {x[3 * i], x[3 * i + 1], x[3 * i + 2], (double)t};
    S.pos[i] = V3{p.x, p.y, p.z};
    S.typ[i] = (uint8_t)(t | (S.bstart[i + 1] > S.bstart[i] ? TYP_BONDED : 0));   // bonds by caller id = i
    S.xb[i] = F3{(float)p.x, (float)p.y, (float)p.z};
    S.xp[i] = S.xb[i];
    S.vel[i] = V3{v[3 * i], v[3 * i + 1], v[3 * i + 2]};
    if (t == 0) {
        S.ori[i] = V3{n[3 * i], n[3 * i + 1], n[3 * i + 2]};
        S.angv[i] = V3{w[3 * i], w[3 * i + 1], w[3 * i + 2]};
    } else {
        S.ori[i] = V3{0.0, 0.0, 0.0};
        S.angv[i] = V3{0.0, 0.0, 0.0};
    }
    S.frc[i] = V3{0.0, 0.0, 0.0};
    S.trq[i] = V3{0.0, 0.0, 0.0};
    S.gid[i] = i;
    S.slot[i] = i;
    S.owner[i] = -1;
}

__global__ void k_pack_multi(const SysDev *Sd, int s, const double *x, const double *n, const int32_t *type,
                             const double *v, const double *w) {
    pack_one(Sd[s], x, n, type, v, w);
}

// ------------------------------------------------------------------ seeds from lipids

// Seed j < kl starts at the position of lipid number floor(j * N_L / kl) (lipids in
// id order; `lip` lists their ids).  With a separate protein set, seed kl + j
// starts at protein number floor(j * N_P / (k - kl)), whose ids follow the lipids'
// in `lip`.  No warm start for the first assignment.
__global__ void k_init_seeds(const SysDev *Sd, Maps L_maps, const int32_t *const *lipids) {
    SYS_FROM(c);
    if (!S.sc->rebuild) return;
    int c = lb * BLOCK + threadIdx.x;
    if (c < S.k) {
        long long j;
        if (c < S.kl) j = (long long)c * S.nlip / S.kl;
        else j = S.nlip + (long long)(c - S.kl) * S.nsrcp / (S.k - S.kl);
        int g = lipids[s][j];
        D4 p = ld3(S.pos + S.slot[g]);
        p.x = wrap_coord(p.x, S.per[0], S.box[0]);
        p.y = wrap_coord(p.y, S.per[1], S.box[1]);
        p.z = wrap_coord(p.z, S.per[2], S.box[2]);
        p.w = 0.0;
        S.seed[c] = p;
    }
}

// ------------------------------------------------------------------ seed grid

// Per-block bounding boxes of the (wrapped) particle positions: partials 2..7 of bred2
// (bred holds the statistics of the last drift, which the next step kernel publishes).
__global__ __launch_bounds__(BLOCK) void k_bbox_partial(const SysDev *Sd, Maps L_maps) {
    SYS_FROM(p);
    if (!S.sc->rebuild) return;
    __shared__ double s_v[6][BLOCK / WAVE];
    const int i = lb * BLOCK + threadIdx.x;
    double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (i < S.n) {
        D4 p = ld3(S.pos + i);
        double v[3] = {wrap_coord(p.x, S.per[0], S.box[0]), wrap_coord(p.y, S.per[1], S.box[1]),
                       wrap_coord(p.z, S.per[2], S.box[2])};
        for (int a = 0; a < 3; ++a) { mn[a] = v[a]; mx[a] = v[a]; }
    }
    for (int a = 0; a < 3; ++a) {
        mn[a] = wave_min(mn[a]);
        mx[a] = wave_max(mx[a]);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == WAVE - 1)
        for (int a = 0; a < 3; ++a) { s_v[a][w] = mn[a]; s_v[3 + a][w] = mx[a]; }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int a = threadIdx.x;
        double r = s_v[a][0];
        for (int q = 1; q < BLOCK / WAVE; ++q) r = (a < 3) ? fmin(r, s_v[a][q]) : fmax(r, s_v[a][q]);
        S.bred2[(size_t)lb * BRED + 2 + a] = r;
    }
}

// Per-block bounding boxes of the seeds (unwrapped centroids), 256 seeds per block.
__global__ __launch_bounds__(BLOCK) void k_seed_bbox_partial(const SysDev *Sd, Maps L_maps) {
    SYS_FROM(c);
    if (!S.sc->rebuild) return;
    __shared__ double s_v[6][BLOCK / WAVE];
    const int c = lb * BLOCK + threadIdx.x;
    double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    if (c < S.k) {
        const D4 p = S.seed[c];
        const double v[3] = {p.x, p.y, p.z};
        for (int a = 0; a < 3; ++a) { mn[a] = v[a]; mx[a] = v[a]; }
    }
    for (int a = 0; a < 3; ++a) {
        mn[a] = wave_min(mn[a]);
        mx[a] = wave_max(mx[a]);
    }
    const int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == WAVE - 1)
        for (int a = 0; a < 3; ++a) { s_v[a][w] = mn[a]; s_v[3 + a][w] = mx[a]; }
    __syncthreads();
    if (threadIdx.x < 6) {
        const int a = threadIdx.x;
        double r = s_v[a][0];
        for (int q = 1; q < BLOCK / WAVE; ++q) r = (a < 3) ? fmin(r, s_v[a][q]) : fmax(r, s_v[a][q]);
        S.sbox[(size_t)lb * 6 + a] = r;
    }
}

// Bounding boxes and grid geometry, one block per system (from the per-block partials).
// Uniform grid over the seeds: cubic cells holding about one eighth of a seed each,
// but no smaller than hmin (twice the cell-pair search radius).  A cell-pair query
// walks every grid cell within its reach; on small systems a finer grid would make
// each query a long chain of dependent loads over mostly empty cells.  The seeds' boxes are
// sper to a 256-cell block of the cell map.
__global__ __launch_bounds__(1024) void k_grid_setup(const SysDev *Sd, int nsys, double hmin, int sper) {
    const SysDev &S = Sd[blockIdx.x];
    if (!S.sc->rebuild) return;
    __shared__ double s_mn[6][16], s_mx[6][16];
    double mn[6], mx[6];
    for (int a = 0; a < 6; ++a) { mn[a] = INFINITY; mx[a] = -INFINITY; }
    const int nblk = (S.n + BLOCK - 1) / BLOCK;
    for (int b = threadIdx.x; b < nblk; b += blockDim.x) {
        const double *r = S.bred2 + (size_t)b * BRED + 2;
        for (int a = 0; a < 3; ++a) { mn[a] = fmin(mn[a], r[a]); mx[a] = fmax(mx[a], r[3 + a]); }
    }
    const int nsb = sper * ((S.k + BLOCK - 1) / BLOCK);
    for (int b = threadIdx.x; b < nsb; b += blockDim.x) {
        const double *r = S.sbox + (size_t)b * 6;
        for (int a = 0; a < 3; ++a) { mn[3 + a] = fmin(mn[3 + a], r[a]); mx[3 + a] = fmax(mx[3 + a], r[3 + a]); }
    }
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int a = 0; a < 6; ++a) {
        mn[a] = wave_min(mn[a]);
        mx[a] = wave_max(mx[a]);
        if (lane == WAVE - 1) { s_mn[a][w] = mn[a]; s_mx[a][w] = mx[a]; }
    }
    __syncthreads();
    if (w != 0) return;
    for (int a = 0; a < 6; ++a) {                    // sixteen wavefronts: a row of lanes
        mn[a] = row_min(s_mn[a][lane & 15]);
        mx[a] = row_max(s_mx[a][lane & 15]);
    }
    if (lane == 15) {
        SysScal *sc = S.sc;
        double ext[3];
        for (int a = 0; a < 3; ++a) {
            // seed box for Morton keys: the box on periodic axes, the seeds' extent otherwise
            sc->slo[a] = S.per[a] ? 0.0 : mn[3 + a];
            sc->shi[a] = S.per[a] ? S.box[a] : mx[3 + a];
            if (S.per[a]) {
                sc->glo[a] = 0.0;
                ext[a] = S.box[a];
            } else {
                double lo = fmin(mn[a], mn[3 + a]), hi = fmax(mx[a], mx[3 + a]);
                if (!(lo <= hi)) { lo = 0.0; hi = 0.0; }
                double pad = 1e-6 * (hi - lo) + 1e-6;
                sc->glo[a] = lo - pad;
                ext[a] = (hi - lo) + 2.0 * pad;
            }
        }
        double cap = (double)max(1, S.gcap);
        double vol = fmax(ext[0], 1.0) * fmax(ext[1], 1.0) * fmax(ext[2], 1.0);
        double h = fmax(hmin, cbrt(vol / cap));
        int dims[3];
        for (int it = 0; it < 200; ++it) {
            double prod = 1.0;
            for (int a = 0; a < 3; ++a) {
                if (S.per[a]) dims[a] = max(1, (int)floor(ext[a] / h));
                else dims[a] = max(1, (int)ceil(ext[a] / h));
                prod *= dims[a];
            }
            if (prod <= cap) break;
            h *= 1.1;
        }
        if ((double)dims[0] * dims[1] * dims[2] > cap || !isfinite(h)) {
            dims[0] = dims[1] = dims[2] = 1;
            h = fmax(ext[0], fmax(ext[1], ext[2]));
            if (!isfinite(h) || !(h > 0.0)) h = 1.0;
        }
        for (int a = 0; a < 3; ++a) {
            sc->gdim[a] = dims[a];
            sc->gh[a] = S.per[a] ? ext[a] / dims[a] : h;
        }
        sc->gtot = dims[0] * dims[1] * dims[2];
    }
}

__device__ __forceinline__ int grid_coord(const SysScal *sc, const SysDev &S, int a, double v, double &u) {
    u = wrap_coord(v, S.per[a], S.box[a]) - sc->glo[a];
    int c = (int)floor(u / sc->gh[a]);
    c = max(0, min(c, sc->gdim[a] - 1));
    return c;
}

// (gcount is zero between grid builds: the fill takes back what the count adds.)
__global__ void k_grid_count(const SysDev *Sd, Maps L_maps) {
    SYS_FROM(c);
    if (!S.sc->rebuild) return;
    int c = lb * BLOCK + threadIdx.x;
    if (c >= S.k) return;
    const SysScal *sc = S.sc;
    D4 p = S.seed[c];
    double u;
    int gx = grid_coord(sc, S, 0, p.x, u), gy = grid_coord(sc, S, 1, p.y, u), gz = grid_coord(sc, S, 2, p.z, u);
    int g = (gx * sc->gdim[1] + gy) * sc->gdim[2] + gz;
    S.sgcell[c] = g;
    atomicAdd(&S.gcount[g], 1);
}

// Segmented exclusive scans, three launches (tile sums, per-system scan of the
// tile sums, tile scans), specialised at compile time per array.  WHICH: 0 = seed
// grid (gcount -> gstart over gtot cells), 1 = ccount2 -> cstart2, 2 = ccount2 ->
// cstart, the counts moving to ccount, 3 = cnbr_start in place (k cells).  dst[len]
// receives the total.
template <int WHICH>
__device__ __forceinline__ const int *scan_src(const SysDev &S) {
    if constexpr (WHICH == 0) return S.gcount;
    else if constexpr (WHICH == 1 || WHICH == 2) return S.ccount2;
    else return S.cnbr_start;
}
template <int WHICH>
__device__ __forceinline__ int *scan_dst(const SysDev &S) {
    if constexpr (WHICH == 0) return S.gstart;
    else if constexpr (WHICH == 1) return S.cstart2;
    else if constexpr (WHICH == 2) return S.cstart;
    else return S.cnbr_start;
}
template <int WHICH>
__device__ __forceinline__ int scan_len(const SysDev &S) {
    if constexpr (WHICH == 0) return S.sc->gtot;
    else return S.k;
}

template <int WHICH>
__global__ __launch_bounds__(BLOCK) void k_scan_a(const SysDev *Sd, Maps L_maps) {
    const int32_t *map = WHICH == 0 ? L_maps.sg : L_maps.sc;
    const int s = find_sys(map, L_maps.nsys, blockIdx.x);
    const SysDev &S = Sd[s];
    if (!S.sc->rebuild) return;
    const int tile = blockIdx.x - map[s];
    const int *src = scan_src<WHICH>(S);
    const int len = scan_len<WHICH>(S);
    __shared__ int s_w[16];
    constexpr int per = SCAN_TILE / BLOCK;
    int loc = 0;
    for (int q = 0; q < per; ++q) {
        const int idx = tile * SCAN_TILE + threadIdx.x * per + q;
        if (idx < len) loc += src[idx];
    }
    int tot;
    (void)block_excl_scan(loc, s_w, tot);
    if (threadIdx.x == 0) S.tsum[tile] = tot;
}

template <int WHICH>
__global__ __launch_bounds__(1024) void k_scan_b(const SysDev *Sd) {
    const SysDev &S = Sd[blockIdx.x];
    if (!S.sc->rebuild) return;
    __shared__ int s_w[16];
    const int ntile = (scan_len<WHICH>(S) + SCAN_TILE - 1) / SCAN_TILE;
    block_scan_array(S.tsum, ntile, s_w);
}

template <int WHICH>
__global__ __launch_bounds__(BLOCK) void k_scan_c(const SysDev *Sd, Maps L_maps) {
    const int32_t *map = WHICH == 0 ? L_maps.sg : L_maps.sc;
    const int s = find_sys(map, L_maps.nsys, blockIdx.x);
    const SysDev &S = Sd[s];
    if (!S.sc->rebuild) return;
    const int tile = blockIdx.x - map[s];
    const int *src = scan_src<WHICH>(S);
    int *dst = scan_dst<WHICH>(S);
    const int len = scan_len<WHICH>(S);
    const int ntile = (len + SCAN_TILE - 1) / SCAN_TILE;
    if (tile >= ntile) return;
    __shared__ int s_w[16];
    constexpr int per = SCAN_TILE / BLOCK;
    int v[per];
    int loc = 0;
    for (int q = 0; q < per; ++q) {
        const int idx = tile * SCAN_TILE + threadIdx.x * per + q;
        v[q] = (idx < len) ? src[idx] : 0;
        loc += v[q];
    }
    int tot;
    int run = S.tsum[tile] + block_excl_scan(loc, s_w, tot);
    for (int q = 0; q < per; ++q) {
        const int idx = tile * SCAN_TILE + threadIdx.x * per + q;
        if (idx < len) {
            dst[idx] = run;
            if constexpr (WHICH == 2) {
                S.ccount[idx] = v[q];
                S.ccount2[idx] = 0;
            }
        }
        run += v[q];
    }
    if (tile == ntile - 1 && threadIdx.x == 0) dst[len] = S.tsum[ntile];
}

// The whole scan of a system by one block, up to SCAN_ONE elements (64 per thread): one
// launch of 4.5 us instead of three of 10 us together at 50 thousand grid cells.  Beyond
// SCAN_ONE one block's rounds take longer than the three launches.
constexpr int SCAN_ONE = 65536;

template <int WHICH>
__global__ __launch_bounds__(1024) void k_scan_one(const SysDev *Sd) {
    const SysDev &S = Sd[blockIdx.x];
    if (S.n <= 0 || !S.sc->rebuild) return;
    __shared__ int s_w[16];
    const int *src = scan_src<WHICH>(S);
    int *dst = scan_dst<WHICH>(S);
    const int len = scan_len<WHICH>(S);
    // eight consecutive elements per thread and round, in 16-byte accesses (the arrays start
    // on 256 bytes); the next round's are on their way while this one is scanned
    constexpr int PER = 8, Q = PER / 4;
    typedef int v4i __attribute__((ext_vector_type(4)));
    auto load = [&](int i0, v4i (&v)[Q]) {
#pragma unroll
        for (int h = 0; h < Q; ++h) {
            const int i = i0 + 4 * h;
            if (i + 3 < len) v[h] = ldg(reinterpret_cast<const v4i *>(src + i));
            else v[h] = v4i{i < len ? ldg(src + i) : 0, i + 1 < len ? ldg(src + i + 1) : 0, i + 2 < len ? ldg(src + i + 2) : 0, 0};
        }
    };
    auto store = [&](int *p, int i0, const v4i (&v)[Q]) {
#pragma unroll
        for (int h = 0; h < Q; ++h) {
            const int i = i0 + 4 * h;
            if (i + 3 < len) stg(reinterpret_cast<v4i *>(p + i), v[h]);
            else
                for (int q = 0; q < 3; ++q)
                    if (i + q < len) stg(p + i + q, q == 0 ? v[h].x : (q == 1 ? v[h].y : v[h].z));
        }
    };
    int carry = 0;
    v4i nx[Q];
    load((int)threadIdx.x * PER, nx);
    for (int base = 0; base < len; base += 1024 * PER) {
        const int i0 = base + (int)threadIdx.x * PER;
        v4i v[Q], out[Q];
        int loc = 0;
#pragma unroll
        for (int h = 0; h < Q; ++h) {
            v[h] = nx[h];
            loc += v[h].x + v[h].y + v[h].z + v[h].w;
        }
        load(i0 + 1024 * PER, nx);
        int tot;
        int run = carry + block_excl_scan(loc, s_w, tot);
#pragma unroll
        for (int h = 0; h < Q; ++h)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                out[h][q] = run;
                run += v[h][q];
            }
        store(dst, i0, out);
        if constexpr (WHICH == 2) {
            const v4i zero[Q] = {};
            store(S.ccount, i0, v);
            store(S.ccount2, i0, zero);
        }
        carry += tot;
    }
    if (threadIdx.x == 0) dst[len] = carry;
}

template <int WHICH>
static void launch_scan_t(const LaunchCtx &L) {
    if ((WHICH == 0 ? L.gmax : L.kmax) <= SCAN_ONE) {
        hipLaunchKernelGGL(k_scan_one<WHICH>, dim3(L.nsys), dim3(1024), 0, L.st, L.S);
        return;
    }
    const int nblk = WHICH == 0 ? L.nblk_sg : L.nblk_sc;
    hipLaunchKernelGGL(k_scan_a<WHICH>, dim3(nblk), dim3(BLOCK), 0, L.st, L.S, L.maps);
    hipLaunchKernelGGL(k_scan_b<WHICH>, dim3(L.nsys), dim3(1024), 0, L.st, L.S);
    hipLaunchKernelGGL(k_scan_c<WHICH>, dim3(nblk), dim3(BLOCK), 0, L.st, L.S, L.maps);
}

static void launch_scan(const LaunchCtx &L, int which) {
    switch (which) {
        case 0: launch_scan_t<0>(L); break;
        case 1: launch_scan_t<1>(L); break;
        case 2: launch_scan_t<2>(L); break;
        default: launch_scan_t<3>(L); break;
    }
}

__global__ void k_grid_fill(const SysDev *Sd, Maps L_maps) {
    SYS_FROM(c);
    if (!S.sc->rebuild) return;
    int c = lb * BLOCK + threadIdx.x;
    if (c >= S.k) return;
    int g = S.sgcell[c];
    int p = S.gstart[g] + atomicAdd(&S.gcount[g], -1) - 1;
    S.val2[p] = (uint32_t)c;
}

// Seeds inside a grid cell in ascending index order (deterministic scans): each seed's place
// is the number of smaller ones in its cell.  With the centroid positions in grid order,
// seed index in w (one load per candidate in the E-step).
__global__ void k_grid_place(const SysDev *Sd, Maps L_maps) {
    SYS_FROM(c);
    if (!S.sc->rebuild) return;
    const int c = lb * BLOCK + threadIdx.x;
    if (c >= S.k) return;
    const int g = S.sgcell[c], b = S.gstart[g], e = S.gstart[g + 1];
    int at = b;
    for (int q = b; q < e; ++q) at += (int)ldg(reinterpret_cast<const int32_t *>(S.val2) + q) < c ? 1 : 0;
    const D4 p = S.seed[c];
    S.gseed[at] = c;
    S.gpos[at] = D4{p.x, p.y, p.z, (double)c};
}

// The particles do not move while the cells update: their boxes serve all of its grids.
void launch_particle_boxes(const LaunchCtx &L) {
    hipLaunchKernelGGL(k_bbox_partial, dim3(L.nblk_p), dim3(BLOCK), 0, L.st, L.S, L.maps);
}

static void grid_build(const LaunchCtx &L, int sper) {
    hipLaunchKernelGGL(k_grid_setup, dim3(L.nsys), dim3(1024), 0, L.st, L.S, L.nsys, 2.0 * L.prm.cell_search, sper);
    hipLaunchKernelGGL(k_grid_count, dim3(L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps);
    launch_scan(L, 0);
    hipLaunchKernelGGL(k_grid_fill, dim3(L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps);
    hipLaunchKernelGGL(k_grid_place, dim3(L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps);
}

// ------------------------------------------------------------------ E-step

// Per-axis window of grid offsets searched at radius r: open axes are clipped at
// the grid edge, periodic axes stop growing once every cell is covered.
__device__ __forceinline__ void axis_window(int c, int dim, int per, int r, int &lo, int &hi) {
    if (per) {
        int half = (dim - 1) / 2;
        lo = -min(r, half);
        hi = min(r, dim - 1 - half);
    } else {
        lo = max(-r, -c);
        hi = min(r, dim - 1 - c);
    }
}

// Nearest centroid among seeds [slo, shi) (ties: lower index).  ranges: nine entries of LDS
// for this thread, BLOCK apart.
__device__ __forceinline__ int nearest_seed(const SysDev &S, const SysScal *sc, double xi, double yi, double zi, int warm,
                                            int slo, int shi, int2 *ranges, double &bestd2) {
    int best = -1;
    bestd2 = INFINITY;
    double dx, dy, dz;
    const unsigned span = (unsigned)(shi - slo);
    if (warm >= 0 && (unsigned)(warm - slo) < span) {
        D4 c = S.seed[warm];
        bestd2 = dist2_exact(S, xi, yi, zi, c.x, c.y, c.z, dx, dy, dz);
        best = warm;
    }
    double u[3];
    int cc[3];
    cc[0] = grid_coord(sc, S, 0, xi, u[0]);
    cc[1] = grid_coord(sc, S, 1, yi, u[1]);
    cc[2] = grid_coord(sc, S, 2, zi, u[2]);
    int plo[3] = {1, 1, 1}, phi[3] = {-1, -1, -1};
    int rmax = max(sc->gdim[0], max(sc->gdim[1], sc->gdim[2]));
    // whether every seed outside the window [lo, hi] is farther than the best one: compares it
    // with the distance from the particle to the nearest cell not yet visited
    auto done = [&](const int (&lo)[3], const int (&hi)[3]) {
        double m = INFINITY;
        for (int a = 0; a < 3; ++a) {
            int dim = sc->gdim[a];
            bool full = S.per[a] ? (hi[a] - lo[a] + 1 >= dim) : false;
            if (full) continue;
            bool lo_open = S.per[a] ? true : (cc[a] + lo[a] > 0);
            bool hi_open = S.per[a] ? true : (cc[a] + hi[a] < dim - 1);
            if (lo_open) m = fmin(m, u[a] - (double)(cc[a] + lo[a]) * sc->gh[a]);
            if (hi_open) m = fmin(m, (double)(cc[a] + hi[a] + 1) * sc->gh[a] - u[a]);
        }
        if (m == INFINITY) return true;
        if (best >= 0 && m > 0.0) {
            double mm = m * (1.0 - 1e-9);
            if (bestd2 < mm * mm) return true;
        }
        return false;
    };
    // The cells around the particle's own first, at once: nine columns of three grid cells,
    // less what is farther away than the warm start (which leaves one to four), whose seed
    // ranges are all loaded together; then their seeds, own column first.  Nearly every
    // particle ends here.  The widening search below takes what does not (it is a chain of
    // dependent loads), and the windows that wrap along z or cover a whole periodic axis.
    int r0 = 0;
    {
        const bool zin = !S.per[2] || (cc[2] >= 1 && cc[2] + 1 < sc->gdim[2]);
        if (zin && !(S.per[0] && sc->gdim[0] < 3) && !(S.per[1] && sc->gdim[1] < 3)) {
            int lo[3], hi[3];
            double gap2[3][3];                       // squared distance to the rows at -1, 0, 1 along each axis
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                axis_window(cc[a], sc->gdim[a], S.per[a], 1, lo[a], hi[a]);
                const double gl = fmax(u[a] - (double)cc[a] * sc->gh[a] - 1e-9, 0.0);
                const double gr = fmax((double)(cc[a] + 1) * sc->gh[a] - u[a] - 1e-9, 0.0);
                gap2[a][0] = gl * gl * (1.0 - 1e-9);
                gap2[a][1] = 0.0;
                gap2[a][2] = gr * gr * (1.0 - 1e-9);
            }
            const int zlo = gap2[2][0] > bestd2 ? 0 : lo[2], zhi = gap2[2][2] > bestd2 ? 0 : hi[2];
            constexpr int NC = 9;
            constexpr int ord[NC] = {4, 1, 3, 5, 7, 0, 2, 6, 8};
            int qb[NC], qe[NC];
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                const int ox = ord[k] / 3 - 1, oy = ord[k] % 3 - 1;
                const bool in = ox >= lo[0] && ox <= hi[0] && oy >= lo[1] && oy <= hi[1] &&
                                !(gap2[0][ox + 1] + gap2[1][oy + 1] > bestd2);
                int gx = cc[0] + ox, gy = cc[1] + oy;
                if (S.per[0]) gx = gx < 0 ? gx + sc->gdim[0] : (gx >= sc->gdim[0] ? gx - sc->gdim[0] : gx);
                if (S.per[1]) gy = gy < 0 ? gy + sc->gdim[1] : (gy >= sc->gdim[1] ? gy - sc->gdim[1] : gy);
                const int base = (gx * sc->gdim[1] + gy) * sc->gdim[2] + cc[2];
                qb[k] = in ? ldg(S.gstart + base + zlo) : 0;
                qe[k] = in ? ldg(S.gstart + base + zhi + 1) : 0;
            }
            int nr = 0;
#pragma unroll
            for (int k = 0; k < NC; ++k)
                if (qe[k] > qb[k]) ranges[nr++ * BLOCK] = make_int2(qb[k], qe[k]);
            // each lane goes through its own ranges, whatever the others' lengths
            auto columns = [&](auto per_tag) {
                constexpr bool PER = decltype(per_tag)::value;
                constexpr int SB = 2;                // seeds side by side
                int2 r = nr > 0 ? ranges[0] : make_int2(0, 0);
                int k = 1;
                while (r.x < r.y) {
                    D4 c[SB];
#pragma unroll
                    for (int h = 0; h < SB; ++h) c[h] = ldg(S.gpos + min(r.x + h, r.y - 1));
                    r.x += SB;
                    if (r.x >= r.y && k < nr) r = ranges[k++ * BLOCK];
#pragma unroll
                    for (int h = 0; h < SB; ++h) {
                        const int sd = (int)c[h].w;
                        const double d2 = PER ? dist2_exact(S, xi, yi, zi, c[h].x, c[h].y, c[h].z, dx, dy, dz)
                                              : dist2_open(xi, yi, zi, c[h].x, c[h].y, c[h].z, dx, dy, dz);
                        // (not the other particle set's cells)
                        if ((unsigned)(sd - slo) < span && (d2 < bestd2 || (d2 == bestd2 && sd < best))) {
                            bestd2 = d2;
                            best = sd;
                        }
                    }
                }
            };
            if ((S.per[0] | S.per[1] | S.per[2]) != 0) columns(std::true_type{});
            else columns(std::false_type{});
            if (done(lo, hi)) return best;
            for (int a = 0; a < 3; ++a) { plo[a] = lo[a]; phi[a] = hi[a]; }
            r0 = 2;
        }
    }
    for (int r = r0; r <= rmax; ++r) {
        int lo[3], hi[3];
        bool grew = false;
        for (int a = 0; a < 3; ++a) {
            axis_window(cc[a], sc->gdim[a], S.per[a], r, lo[a], hi[a]);
            if (lo[a] < plo[a] || hi[a] > phi[a]) grew = true;
        }
        if (!grew) break;   // every cell visited
        for (int ox = lo[0]; ox <= hi[0]; ++ox) {
            bool nx = (ox < plo[0] || ox > phi[0]);
            int gx = cc[0] + ox;
            if (S.per[0]) gx = (gx % sc->gdim[0] + sc->gdim[0]) % sc->gdim[0];
            for (int oy = lo[1]; oy <= hi[1]; ++oy) {
                bool ny = nx || (oy < plo[1] || oy > phi[1]);
                int gy = cc[1] + oy;
                if (S.per[1]) gy = (gy % sc->gdim[1] + sc->gdim[1]) % sc->gdim[1];
                // the column's cells not visited at a smaller radius: the whole z window
                // where the column is new, else the rows below and above the previous
                // window; each a run of consecutive grid cells (split where a periodic z
                // axis wraps), whose seeds are one range of gpos
                int ra[2], rb[2], nr = 0;
                if (ny) {
                    ra[0] = lo[2]; rb[0] = hi[2]; nr = 1;
                } else {
                    if (lo[2] < plo[2]) { ra[nr] = lo[2]; rb[nr] = min(hi[2], plo[2] - 1); ++nr; }
                    if (hi[2] > phi[2]) { ra[nr] = max(lo[2], phi[2] + 1); rb[nr] = hi[2]; ++nr; }
                }
                const int nzg = sc->gdim[2], base = (gx * sc->gdim[1] + gy) * nzg;
                for (int k = 0; k < nr; ++k) {
                    int za = cc[2] + ra[k], zb = cc[2] + rb[k];
                    int z2a = 0, z2b = -1;                // the wrapped part, if any
                    if (S.per[2]) {                       // the window spans at most nzg rows
                        if (za < 0) {
                            if (zb < 0) { za += nzg; zb += nzg; }
                            else { z2a = 0; z2b = zb; za += nzg; zb = nzg - 1; }
                        } else if (zb >= nzg) {
                            if (za >= nzg) { za -= nzg; zb -= nzg; }
                            else { z2a = 0; z2b = zb - nzg; zb = nzg - 1; }
                        }
                    }
                    for (int part = 0; part < 2; ++part) {
                        const int a0 = part ? z2a : za, a1 = part ? z2b : zb;
                        if (a1 < a0) continue;
                        const int qe = ldg(S.gstart + base + a1 + 1);
                        for (int q = ldg(S.gstart + base + a0); q < qe; ++q) {
                            const D4 c = ldg(S.gpos + q);
                            const int sd = (int)c.w;
                            if ((unsigned)(sd - slo) >= span) continue;   // the other particle set's cells
                            double d2 = dist2_exact(S, xi, yi, zi, c.x, c.y, c.z, dx, dy, dz);
                            if (d2 < bestd2 || (d2 == bestd2 && sd < best)) { bestd2 = d2; best = sd; }
                        }
                    }
                }
            }
        }
        for (int a = 0; a < 3; ++a) { plo[a] = lo[a]; phi[a] = hi[a]; }
        if (done(lo, hi)) break;
    }
    return best;
}

// The order in which iteration `it` of an update goes through the particles: their slots
// at first, then cell by cell.  The iterations reorder only what they need (positions,
// types and slots), in memory that is idle until the update moves the particles.
struct Order {
    V3 *pos;
    uint8_t *typ;
    uint32_t *idx;                                  // slots (null: the order is the slots')
};
__device__ __forceinline__ Order order_of(const SysDev &S, int it) {
    if (it == 0) return Order{S.pos, S.typ, nullptr};
    if (it & 1) return Order{S.vel2, S.typ2, reinterpret_cast<uint32_t *>(S.frc)};
    return Order{S.ori2, reinterpret_cast<uint8_t *>(S.angv2), reinterpret_cast<uint32_t *>(S.trq)};
}

// The nearest centroid of each particle, and its place among the cell's members: one atomic
// per run of neighbouring lanes with the same cell.  (Places within a cell are put in order
// by k_centroids.)  Bound by its chain of dependent loads on small systems (125k particles:
// 43.6 us with the widening search alone, 26.9 with the nine columns loaded together, 19.1
// with each lane on its own ranges) and by vector instructions, about 23 per candidate, on
// large ones (4M, a fresh cell: 476, 359 and 238 us; 213 once it has run).
__global__ __launch_bounds__(BLOCK) void k_assign(const SysDev *Sd, Maps L_maps, int it, int warm) {
    SYS_FROM(p);
    if (!S.sc->rebuild) return;
    __shared__ int2 s_r[9 * BLOCK];
    const int j = lb * BLOCK + threadIdx.x, lane = threadIdx.x & (WAVE - 1);
    int best = -1;
    if (j < S.n) {
        const Order o = order_of(S, it);
        const V3 p = ldg(o.pos + j);
        double d2;
        // lipids search cells [0, kl), protein beads [kl, k) (all cells when kl == k)
        const bool lipid_set = (ldg(o.typ + j) & TYP_MASK) == 0 || S.kl == S.k;
        const int slo = lipid_set ? 0 : S.kl, shi = lipid_set ? S.kl : S.k;
        best = nearest_seed(S, S.sc, p.x, p.y, p.z, warm ? S.owner[j] : -1, slo, shi, s_r + threadIdx.x, d2);
        if (best < 0) { atomicOr(&S.sc->err, ERR_ASSIGN); best = 0; }
    }
    const int prev = __shfl_up(best, 1);
    const unsigned long long heads = __ballot(lane == 0 || best != prev);
    const int head = 63 - __clzll(heads & (~0ull >> (63 - lane)));
    const unsigned long long later = lane == 63 ? 0ull : heads & (~0ull << (lane + 1));
    int base = 0;
    if (lane == head && best >= 0) base = atomicAdd(S.ccount2 + best, (later ? __ffsll(later) - 1 : WAVE) - lane);
    base = __shfl(base, head);
    if (best >= 0) S.key[j] = (uint64_t)(unsigned)best | (uint64_t)(unsigned)(base + lane - head) << 32;
}

__global__ __launch_bounds__(BLOCK) void k_cell_place(const SysDev *Sd, Maps L_maps) {
    SYS_FROM(p);
    if (!S.sc->rebuild) return;
    const int j = lb * BLOCK + threadIdx.x;
    if (j >= S.n) return;
    const uint64_t key = S.key[j];
    S.val[S.cstart[(int)(key & 0xffffffffu)] + (int)(key >> 32)] = (uint32_t)j;
}

// ------------------------------------------------------------------ M-step

// CELL_LANES lanes per cell, CB_BLOCKS blocks per 256-cell block of the cell map.  The
// members are put in the iteration's order by counting, among a cell's, those before each;
// their offsets from the centroid wait in LDS for the sum, which is taken in that order.
// Each centroid with lipid members moves by the mean min-image offset of those members;
// centroids without lipids stay; periodic axes wrap.  Cells of a separate protein set
// (index >= kl) average their protein members.  The members go on in their new order
// (k_assign's next iteration), and each block leaves its centroids' box.
//  What bounds it is the latency of one chain (members, their positions, the sum).  This and
// the assignment's counts replaced a radix sort of the particles by cell (two passes of three
// launches), the gather of the whole state, the cell ranges and a serial sum per thread:
// 12.5 us, with 8 for the counts' scan and placing, instead of 104 at 125k particles.
//  A cell of more than CMEM members is left to the whole block: up to BIGS members are
// counted in LDS; the members of a larger one are collected by going through all particles.
// Where cells are that large on average (LaunchCtx::wide), each has a block of its own.
constexpr int CB_BLOCKS = CELL_LANES;
constexpr int CPB = BLOCK / CELL_LANES;            // cells per block
constexpr int CMEM = 64;
constexpr int BIGS = 2048;

// LDS written by one lane and read by others of its wavefront
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Particle j, member `at` of cell `cell` in the new order: its offset from the centroid, 0 if
// it does not count.
__device__ __forceinline__ int centroid_member(const SysDev &S, const Order &o, const Order &w, int last, uint32_t j, int at,
                                               int cell, const D4 &sd, double (&d)[3]) {
    const V3 p = ldg(o.pos + j);
    const uint8_t t = ldg(o.typ + j);
    w.idx[at] = o.idx ? o.idx[j] : j;
    if (!last) {
        w.pos[at] = p;
        w.typ[at] = t;
    }
    S.owner[at] = cell;
    const bool use = ((t & TYP_MASK) == 0) == (cell < S.kl);
    (void)dist2_exact(S, p.x, p.y, p.z, sd.x, sd.y, sd.z, d[0], d[1], d[2]);
    if (!use) d[0] = d[1] = d[2] = 0.0;
    return use ? 1 : 0;
}

// The centroid's coordinate a from the sum of the offsets.
__device__ __forceinline__ double centroid_moved(const SysDev &S, double x, double sum, int cnt, int a) {
#pragma clang fp contract(off)
    if (cnt > 0) {
        x = x + sum / (double)cnt;
        if (S.per[a]) x = x - S.box[a] * floor(x / S.box[a]);
    }
    return x;
}

// A cell's centroid by the whole block, into `out` (LDS) and the system's record.
typedef double CentroidLds[3][CPB * CMEM];         // offsets; a big cell's members, then its offsets
__device__ void centroid_by_block(const SysDev &S, const Order &o, const Order &w, int last, int c, CentroidLds &s_d, int *s_w,
                                  int *s_cnt, double *out, int stride) {
    static_assert(sizeof(s_d) >= 2 * BIGS * sizeof(uint32_t), "a big cell's members");
    const int tid = threadIdx.x, b = S.cstart[c], m = S.ccount[c];
    const D4 sd = S.seed[c];
    if (tid == 0) *s_cnt = 0;
    if (m <= BIGS) {
        uint32_t *s_v = reinterpret_cast<uint32_t *>(s_d);
        for (int q = tid; q < m; q += BLOCK) s_v[q] = S.val[b + q];
        __syncthreads();
        for (int q = tid; q < m; q += BLOCK) {
            const uint32_t v = s_v[q];
            int r = 0;
#pragma unroll 8
            for (int x = 0; x < m; ++x) r += s_v[x] < v ? 1 : 0;
            s_v[BIGS + r] = v;
        }
        __syncthreads();
        for (int q = tid; q < m; q += BLOCK) S.val[b + q] = s_v[BIGS + q];
    } else {
        // the low words of the keys are the cells; each thread takes KP consecutive particles
        constexpr int KP = 8;
        const uint32_t *cell = reinterpret_cast<const uint32_t *>(S.key);
        int at = b;
        for (int j0 = 0; j0 < S.n; j0 += KP * BLOCK) {
            const int jb = j0 + tid * KP;
            unsigned in = 0u;
#pragma unroll
            for (int q = 0; q < KP; ++q)
                if (jb + q < S.n && ldg(cell + 2 * (size_t)(jb + q)) == (uint32_t)c) in |= 1u << q;
            int tot;
            int e = at + block_excl_scan(__popc(in), s_w, tot);
            for (; in; in &= in - 1u) S.val[e++] = (uint32_t)(jb + __ffs(in) - 1);
            at += tot;
        }
    }
    __syncthreads();
    double sum = 0.0;
    int cnt = 0;
    for (int q0 = 0; q0 < m; q0 += BLOCK) {
        if (q0 + tid < m) {
            double d[3];
            cnt += centroid_member(S, o, w, last, S.val[b + q0 + tid], b + q0 + tid, c, sd, d);
            for (int a = 0; a < 3; ++a) s_d[a][tid] = d[a];
        }
        __syncthreads();
        if (tid < 3) {
            const int e = min(BLOCK, m - q0);
#pragma unroll 8
            for (int q = 0; q < e; ++q) sum += s_d[tid][q];
        }
        __syncthreads();
    }
    atomicAdd(s_cnt, cnt);
    __syncthreads();
    if (tid < 3) {
        const double v = centroid_moved(S, tid == 0 ? sd.x : (tid == 1 ? sd.y : sd.z), sum, *s_cnt, tid);
        out[tid * stride] = v;
        reinterpret_cast<double *>(S.seed + c)[tid] = v;
    }
    __syncthreads();
}

__global__ __launch_bounds__(BLOCK) void k_centroids(const SysDev *Sd, Maps L_maps, int it, int last) {
#pragma clang fp contract(off)
    const int cbk = blockIdx.x / CB_BLOCKS;
    const int s = find_sys(L_maps.c, L_maps.nsys, cbk);
    const SysDev &S = Sd[s];
    if (!S.sc->rebuild) return;
    __shared__ CentroidLds s_d;
    __shared__ uint32_t s_j[CPB][CMEM];
    __shared__ int s_big[CPB];
    __shared__ double s_c[3][CPB];
    __shared__ int s_w[16];
    __shared__ int s_cnt;
    const int tid = threadIdx.x, g = tid / CELL_LANES, l = tid % CELL_LANES;
    const int sb = (cbk - L_maps.c[s]) * CB_BLOCKS + blockIdx.x % CB_BLOCKS;     // this block among its system's
    const int c = sb * CPB + g;
    const bool have = c < S.k;
    const Order o = order_of(S, it), w = order_of(S, it + 1);
    const int b = have ? S.cstart[c] : 0, m = have ? S.ccount[c] : 0;
    const D4 sd = S.seed[have ? c : 0];
    if (l == 0) s_big[g] = m > CMEM ? m : 0;
    double mine = l == 0 ? sd.x : (l == 1 ? sd.y : sd.z);      // lanes 0 to 2: the centroid
    if (m <= CMEM) {
        constexpr int R = CMEM / CELL_LANES;
        uint32_t j[R];
        int rk[R] = {0, 0, 0, 0}, cnt = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int q = l + r * CELL_LANES;
            j[r] = q < m ? S.val[b + q] : 0u;
            if (q < m) s_j[g][q] = j[r];
        }
        wave_fence();
        for (int q = 0; q < m; ++q) {
            const uint32_t v = s_j[g][q];
#pragma unroll
            for (int r = 0; r < R; ++r) rk[r] += v < j[r] ? 1 : 0;
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (l + r * CELL_LANES < m) {
                double d[3];
                cnt += centroid_member(S, o, w, last, j[r], b + rk[r], c, sd, d);
                for (int a = 0; a < 3; ++a) s_d[a][g * CMEM + rk[r]] = d[a];
            }
        wave_fence();
        for (int x = 1; x < CELL_LANES; x <<= 1) cnt += __shfl_xor(cnt, x);
        if (l < 3) {
            double sum = 0.0;
#pragma unroll 4
            for (int q = 0; q < m; ++q) sum += s_d[l][g * CMEM + q];
            mine = centroid_moved(S, mine, sum, cnt, l);
        }
    }
    if (l < 3) {
        s_c[l][g] = mine;
        if (have && m <= CMEM) reinterpret_cast<double *>(S.seed + c)[l] = mine;
    }
    __syncthreads();
    for (int h = 0; h < CPB; ++h)
        if (s_big[h]) centroid_by_block(S, o, w, last, sb * CPB + h, s_d, s_w, &s_cnt, &s_c[0][h], CPB);   // block-uniform
    // the block's box (16 centroids: the first row of lanes)
    if (tid < WAVE) {
        const bool in = sb * CPB + (tid & 15) < S.k;
        for (int a = 0; a < 3; ++a) {
            const double lo = row_min(in ? s_c[a][tid & 15] : INFINITY), hi = row_max(in ? s_c[a][tid & 15] : -INFINITY);
            if (tid == 15) {
                S.sbox[(size_t)sb * 6 + a] = lo;
                S.sbox[(size_t)sb * 6 + 3 + a] = hi;
            }
        }
    }
}

// The same with a block per cell (BLOCK of them to a block of the cell map), for large cells.
// The centroids' boxes are taken by k_seed_bbox_partial.
__global__ __launch_bounds__(BLOCK) void k_centroids_wide(const SysDev *Sd, Maps L_maps, int it, int last) {
    const int cbk = blockIdx.x / BLOCK;
    const int s = find_sys(L_maps.c, L_maps.nsys, cbk);
    const SysDev &S = Sd[s];
    if (!S.sc->rebuild) return;
    __shared__ CentroidLds s_d;
    __shared__ double s_c[3];
    __shared__ int s_w[16];
    __shared__ int s_cnt;
    const int c = (cbk - L_maps.c[s]) * BLOCK + blockIdx.x % BLOCK;
    if (c >= S.k) return;
    centroid_by_block(S, order_of(S, it), order_of(S, it + 1), last, c, s_d, s_w, &s_cnt, s_c, 1);
}

// Boxes of the moved centroids to a 256-cell block of the cell map.
static int seed_boxes(const LaunchCtx &L) { return L.wide ? 1 : CB_BLOCKS; }

// One k-means iteration: the seed grid (unless it stands), the particles' cells and the
// centroids' means.
void launch_iteration(const LaunchCtx &L, int it, bool warm, bool last) {
    if (it > 0) grid_build(L, seed_boxes(L));
    hipLaunchKernelGGL(k_assign, dim3(L.nblk_p), dim3(BLOCK), 0, L.st, L.S, L.maps, it, warm ? 1 : 0);
    launch_scan(L, 2);
    hipLaunchKernelGGL(k_cell_place, dim3(L.nblk_p), dim3(BLOCK), 0, L.st, L.S, L.maps);
    if (L.wide) {
        hipLaunchKernelGGL(k_centroids_wide, dim3(BLOCK * L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps, it, last ? 1 : 0);
        hipLaunchKernelGGL(k_seed_bbox_partial, dim3(L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps);
    } else {
        hipLaunchKernelGGL(k_centroids, dim3(CB_BLOCKS * L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps, it, last ? 1 : 0);
    }
}

// ------------------------------------------------------------------ Morton order of centroids

// Segmented stable radix sort of the seeds' 64-bit keys, for launches that hold a system of
// more than RANK_MAX cells.
__global__ __launch_bounds__(BLOCK) void k_sort_hist(const SysDev *Sd, Maps L_maps, int pass) {
    const int32_t *map = L_maps.ts;
    const int s = find_sys(map, L_maps.nsys, blockIdx.x);
    const SysDev &S = Sd[s];
    if (!S.sc->rebuild) return;
    const int tile = blockIdx.x - map[s];
    const int cnt = S.k;
    const uint64_t *keys = (pass & 1) ? S.key2 : S.key;
    const int shift = 8 * pass;
    __shared__ int h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    int base = tile * SORT_TILE;
    for (int r = 0; r < SORT_IPT; ++r) {
        int idx = base + r * BLOCK + threadIdx.x;
        if (idx < cnt) atomicAdd(&h[(int)((keys[idx] >> shift) & 255ull)], 1);
    }
    __syncthreads();
    S.hist[tile * 256 + threadIdx.x] = h[threadIdx.x];
}

// Column scan of the tile histograms: one block per (system, digit) turns the
// digit's per-tile counts into exclusive tile offsets within the digit and leaves
// the digit's total after the last tile row (the scatter adds the digit bases).
__global__ __launch_bounds__(256) void k_sort_scan(const SysDev *Sd) {
    const SysDev &S = Sd[blockIdx.x >> 8];
    if (!S.sc->rebuild) return;
    const int d = blockIdx.x & 255;
    const int cnt = S.k;
    const int ntile = (cnt + SORT_TILE - 1) / SORT_TILE;
    __shared__ int s_w[16];
    int carry = 0;
    for (int t0 = 0; t0 < ntile; t0 += 256) {
        const int t = t0 + (int)threadIdx.x;
        const int v = t < ntile ? S.hist[t * 256 + d] : 0;
        int tot;
        const int ex = block_excl_scan(v, s_w, tot);
        if (t < ntile) S.hist[t * 256 + d] = carry + ex;
        carry += tot;
    }
    if (threadIdx.x == 0) S.hist[ntile * 256 + d] = carry;
}

__global__ __launch_bounds__(BLOCK) void k_sort_scatter(const SysDev *Sd, Maps L_maps, int pass) {
    const int32_t *map = L_maps.ts;
    const int s = find_sys(map, L_maps.nsys, blockIdx.x);
    const SysDev &S = Sd[s];
    if (!S.sc->rebuild) return;
    const int tile = blockIdx.x - map[s];
    const int cnt = S.k;
    const uint64_t *kin = (pass & 1) ? S.key2 : S.key;
    const uint32_t *vin = (pass & 1) ? S.val2 : S.val;
    uint64_t *kout = (pass & 1) ? S.key : S.key2;
    uint32_t *vout = (pass & 1) ? S.val : S.val2;
    const int shift = 8 * pass;
    __shared__ int s_base[256];
    __shared__ int s_cnt[BLOCK / WAVE][256];
    __shared__ int s_w[16];
    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    {
        const int ntile = (cnt + SORT_TILE - 1) / SORT_TILE;
        int tot;
        const int digit_base = block_excl_scan(S.hist[ntile * 256 + tid], s_w, tot);
        s_base[tid] = S.hist[tile * 256 + tid] + digit_base;
    }
    const unsigned long long lt = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
    for (int r = 0; r < SORT_IPT; ++r) {
        for (int q = tid; q < (BLOCK / WAVE) * 256; q += BLOCK) s_cnt[q >> 8][q & 255] = 0;
        __syncthreads();
        int idx = tile * SORT_TILE + r * BLOCK + tid;
        bool valid = idx < cnt;
        uint64_t k = valid ? kin[idx] : 0ull;
        uint32_t v = valid ? vin[idx] : 0u;
        int d = (int)((k >> shift) & 255ull);
        unsigned long long peers = __ballot(valid);
        for (int b = 0; b < 8; ++b) {
            unsigned long long mb = __ballot((d >> b) & 1);
            peers &= ((d >> b) & 1) ? mb : ~mb;
        }
        int rank = __popcll(peers & lt);
        if (valid && rank == 0) s_cnt[w][d] = __popcll(peers);
        __syncthreads();
        if (valid) {
            int pre = 0;
            for (int q = 0; q < w; ++q) pre += s_cnt[q][d];
            int pos = s_base[d] + pre + rank;
            kout[pos] = k;
            vout[pos] = v;
        }
        __syncthreads();
        int add = 0;
        for (int q = 0; q < BLOCK / WAVE; ++q) add += s_cnt[q][tid];
        s_base[tid] += add;
        __syncthreads();
    }
}

static void radix_sort_seeds(const LaunchCtx &L) {
    static_assert(64 % 16 == 0, "an even number of passes: the result lands back in key/val");
    for (int p = 0; p < 64 / 8; ++p) {
        hipLaunchKernelGGL(k_sort_hist, dim3(L.nblk_ts), dim3(BLOCK), 0, L.st, L.S, L.maps, p);
        hipLaunchKernelGGL(k_sort_scan, dim3(L.nsys * 256), dim3(256), 0, L.st, L.S);
        hipLaunchKernelGGL(k_sort_scatter, dim3(L.nblk_ts), dim3(BLOCK), 0, L.st, L.S, L.maps, p);
    }
}

// The seeds' boxes, sper to a 256-cell block of the cell map, into the Morton keys' frame.
__global__ void k_seed_bbox(const SysDev *Sd, int sper) {
    const SysDev &S = Sd[blockIdx.x];
    if (!S.sc->rebuild) return;
    __shared__ double s_mn[3][16], s_mx[3][16];
    double mn[3] = {INFINITY, INFINITY, INFINITY}, mx[3] = {-INFINITY, -INFINITY, -INFINITY};
    const int nsb = sper * ((S.k + BLOCK - 1) / BLOCK);
    for (int b = threadIdx.x; b < nsb; b += blockDim.x) {
        const double *r = S.sbox + (size_t)b * 6;
        for (int a = 0; a < 3; ++a) { mn[a] = fmin(mn[a], r[a]); mx[a] = fmax(mx[a], r[3 + a]); }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        mn[a] = wave_min(mn[a]);
        mx[a] = wave_max(mx[a]);
    }
    int w = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    if (lane == WAVE - 1) for (int a = 0; a < 3; ++a) { s_mn[a][w] = mn[a]; s_mx[a][w] = mx[a]; }
    __syncthreads();
    if (threadIdx.x == WAVE - 1) {
        for (int a = 0; a < 3; ++a) {
            for (int q = 1; q < nw; ++q) { mn[a] = fmin(mn[a], s_mn[a][q]); mx[a] = fmax(mx[a], s_mx[a][q]); }
            S.sc->slo[a] = S.per[a] ? 0.0 : mn[a];
            S.sc->shi[a] = S.per[a] ? S.box[a] : mx[a];
        }
    }
}

// 21-bit quantisation per axis, bits interleaved x (most significant), y, z; bit 63
// marks a protein-set cell, so lipid cells keep the indices below kl.
__global__ void k_morton(const SysDev *Sd, Maps L_maps) {
#pragma clang fp contract(off)
    SYS_FROM(c);
    if (!S.sc->rebuild) return;
    int c = lb * BLOCK + threadIdx.x;
    if (c >= S.k) return;
    D4 p = S.seed[c];
    double v[3] = {p.x, p.y, p.z};
    uint64_t q[3];
    for (int a = 0; a < 3; ++a) {
        double ext = S.sc->shi[a] - S.sc->slo[a];
        if (!(ext > 0.0)) { q[a] = 0; continue; }
        double f = (v[a] - S.sc->slo[a]) / ext;
        double t = floor(f * 2097152.0);
        if (t < 0.0) t = 0.0;
        if (t > 2097151.0) t = 2097151.0;
        q[a] = (uint64_t)t;
    }
    uint64_t key = 0;
    for (int b = 20; b >= 0; --b)
        key = (key << 3) | (((q[0] >> b) & 1ull) << 2) | (((q[1] >> b) & 1ull) << 1) | ((q[2] >> b) & 1ull);
    if (c >= S.kl) key |= 1ull << 63;
    S.key[c] = key;
    S.val[c] = (uint32_t)c;
    S.val2[c] = 0u;
}

// The keys' ranks by comparison, for small systems: each block counts for 256 seeds the
// smaller keys (and the equal ones before them) in one of RANK_SEGS segments.  All k^2
// comparisons take less time than eight radix passes of three launches, whose latency does
// not shrink with the system: 16 us against 230 at 6250 seeds, 80 against 234 at 28 thousand.
// The work grows with the square, so beyond RANK_MAX seeds the radix sort is used.
constexpr int RANK_SEGS = 32;
constexpr int RANK_MAX = 32768;

__global__ __launch_bounds__(BLOCK) void k_rank_seeds(const SysDev *Sd, Maps L_maps) {
    const int cbk = blockIdx.x / RANK_SEGS, seg = blockIdx.x % RANK_SEGS;
    const int s = find_sys(L_maps.c, L_maps.nsys, cbk);
    const SysDev &S = Sd[s];
    if (!S.sc->rebuild) return;
    __shared__ __align__(16) uint64_t s_k[BLOCK];
    const int c0 = (cbk - L_maps.c[s]) * BLOCK, c = c0 + threadIdx.x;
    const uint64_t mine = c < S.k ? S.key[c] : 0ull;
    const int per = (S.k + RANK_SEGS - 1) / RANK_SEGS, b = seg * per, e = min(S.k, b + per);
    int cnt = 0;
    for (int t0 = b; t0 < e; t0 += BLOCK) {
        __syncthreads();
        s_k[threadIdx.x] = t0 + (int)threadIdx.x < e ? S.key[t0 + threadIdx.x] : ~0ull;
        __syncthreads();
        const int m = min(BLOCK, e - t0);
        // a tile wholly before or after this block's seeds needs one comparison per key
        if (t0 + m <= c0) {
#pragma unroll 8
            for (int q = 0; q < m; ++q) cnt += s_k[q] <= mine ? 1 : 0;
        } else if (t0 >= c0 + BLOCK) {
#pragma unroll 8
            for (int q = 0; q < m; ++q) cnt += s_k[q] < mine ? 1 : 0;
        } else {
            for (int q = 0; q < m; ++q) cnt += (s_k[q] < mine || (s_k[q] == mine && t0 + q < c)) ? 1 : 0;
        }
    }
    if (c < S.k && cnt > 0) atomicAdd(S.val2 + c, (uint32_t)cnt);
}

// The cells' new numbers: old cell val[c] becomes c (radix sort), or c becomes val2[c] (ranks).
// cmap[old] = new.
__global__ void k_seed_permute(const SysDev *Sd, Maps L_maps, int ranks) {
    SYS_FROM(c);
    if (!S.sc->rebuild) return;
    int c = lb * BLOCK + threadIdx.x;
    if (c >= S.k) return;
    const int old = ranks ? c : (int)S.val[c], cn = ranks ? (int)S.val2[c] : c;
    S.seed2[cn] = S.seed[old];
    S.ccount2[cn] = S.ccount[old];
    S.cmap[old] = cn;
}

// The particles move to their renumbered cells, in the last iteration's order within a cell,
// CELL_LANES lanes per cell (the whole block for cells of more than CMEM members; with `wide`
// each cell has a block of its own, as in k_centroids_wide).  With the members at hand, each
// cell's radius about its new centroid.  Bound by its scattered reads of whole records (286 us
// at 4M particles, for 0.8 GB of records that make 1.83 GB of traffic).
__global__ __launch_bounds__(BLOCK) void k_move(const SysDev *Sd, Maps L_maps, int iters, int wide) {
    const int per = wide ? BLOCK : CB_BLOCKS;       // blocks to one of the cell map
    const int cbk = blockIdx.x / per;
    const int s = find_sys(L_maps.c, L_maps.nsys, cbk);
    const SysDev &S = Sd[s];
    if (!S.sc->rebuild) return;
    __shared__ int s_big[CPB];
    __shared__ double s_r[BLOCK / WAVE];
    const int tid = threadIdx.x, g = tid / CELL_LANES, l = tid % CELL_LANES;
    const int c0 = ((cbk - L_maps.c[s]) * per + blockIdx.x % per) * (wide ? 1 : CPB), c = c0 + g;
    const bool have = c < S.k && (!wide || g == 0);
    const uint32_t *idx = order_of(S, iters).idx;
    auto one = [&](int from, int to, int cn, const D4 &sd) {
        const uint32_t i = ldg(idx + from);
        const V3 p = ldg(S.pos + i), v = ldg(S.vel + i), n = ldg(S.ori + i), a = ldg(S.angv + i);
        const uint8_t t = ldg(S.typ + i);
        const int32_t id = ldg(S.gid + i);
        S.pos2[to] = p;
        S.vel2[to] = v;
        S.ori2[to] = n;
        S.angv2[to] = a;
        S.typ2[to] = t;
        S.gid2[to] = id;
        S.slot[id] = to;
        S.owner[to] = cn;
        double dx, dy, dz;
        return dist2_exact(S, p.x, p.y, p.z, sd.x, sd.y, sd.z, dx, dy, dz);
    };
    const int b = have ? S.cstart[c] : 0, m = have ? S.ccount[c] : 0;
    const int cn = have ? S.cmap[c] : 0;
    const bool big = have && (wide || m > CMEM);
    if (l == 0) s_big[g] = big ? m : -1;
    double r2 = 0.0;
    if (have && !big) {
        const D4 sd = S.seed[c];
        const int to = S.cstart2[cn];
        for (int q = l; q < m; q += CELL_LANES) r2 = fmax(r2, one(b + q, to + q, cn, sd));
        r2 = row_max(r2);
        if (l == CELL_LANES - 1) S.seed2[cn].w = sqrt(r2);
    }
    __syncthreads();
    for (int h = 0; h < CPB; ++h) {
        const int mb = s_big[h];
        if (mb < 0) continue;                       // block-uniform
        const int cb = c0 + h, cnb = S.cmap[cb], from = S.cstart[cb], to = S.cstart2[cnb];
        const D4 sd = S.seed[cb];
        double rb = 0.0;
        for (int q = tid; q < mb; q += BLOCK) rb = fmax(rb, one(from + q, to + q, cnb, sd));
        rb = wave_max(rb);
        if ((tid & 63) == WAVE - 1) s_r[tid >> 6] = rb;
        __syncthreads();
        rb = fmax(fmax(s_r[0], s_r[1]), fmax(s_r[2], s_r[3]));
        if (tid == 0) S.seed2[cnb].w = sqrt(rb);
        if (tid % CELL_LANES == CELL_LANES - 1) r2 = fmax(r2, rb);
        __syncthreads();
    }
    if (l != CELL_LANES - 1) r2 = 0.0;
    r2 = wave_max(r2);
    if ((tid & 63) == WAVE - 1 && r2 > 0.0) max_if_larger(&S.sc->rmax, dbits(sqrt(r2)));
}

// The renumbered cells become current, and the moved state by swapping its buffer pointers in
// both descriptor tables (the host swaps its copies).
__global__ void k_cell_commit(const SysDev *Sd, Maps L_maps, SysDev *t0, SysDev *t1) {
    SYS_FROM(c);
    if (!S.sc->rebuild) return;
    int c = lb * BLOCK + threadIdx.x;
    if (c >= S.k) return;
    S.seed[c] = S.seed2[c];
    S.ccount[c] = S.ccount2[c];
    S.ccount2[c] = 0;                               // the next assignment counts here
    S.cstart[c] = S.cstart2[c];
    if (c == S.k - 1) S.cstart[S.k] = S.cstart2[S.k];
    if (c < 2) {
        swap_state(c == 0 ? t0[s] : t1[s]);
        if (c == 0 && S.k == 1) swap_state(t1[s]);
    }
}

// Renumber the cells along the Morton curve of their centroids, move the particles, and build
// the new centroids' grid.
void launch_renumber(const LaunchCtx &L, int iters) {
    const bool ranks = L.kmax <= RANK_MAX;
    hipLaunchKernelGGL(k_seed_bbox, dim3(L.nsys), dim3(1024), 0, L.st, L.S, seed_boxes(L));
    hipLaunchKernelGGL(k_morton, dim3(L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps);
    if (ranks) hipLaunchKernelGGL(k_rank_seeds, dim3(RANK_SEGS * L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps);
    else radix_sort_seeds(L);
    hipLaunchKernelGGL(k_seed_permute, dim3(L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps, ranks ? 1 : 0);
    launch_scan(L, 1);
    hipLaunchKernelGGL(k_move, dim3((L.wide ? BLOCK : CB_BLOCKS) * L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps, iters,
                       L.wide ? 1 : 0);
    hipLaunchKernelGGL(k_cell_commit, dim3(L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps, L.tables[0], L.tables[1]);
    grid_build(L, seed_boxes(L));
}

// ------------------------------------------------------------------ cell radii and cell pairs

// The radius of each cell about its centroid, CELL_LANES lanes per cell, for lists rebuilt
// between cell updates (an update's move leaves the radii).  One thread's walk through a
// cell's members is a chain of dependent loads (14.3 us at 125k particles; side by side 10.9
// us, most of it the launch's own chain of map, descriptor, flag and cell loads).
__global__ __launch_bounds__(BLOCK) void k_cell_bounds(const SysDev *Sd, Maps L_maps) {
    const int cbk = blockIdx.x / CB_BLOCKS;
    const int s = find_sys(L_maps.c, L_maps.nsys, cbk);
    const SysDev &S = Sd[s];
    if (!S.sc->rebuild) return;
    const int c = (cbk - L_maps.c[s]) * BLOCK + (blockIdx.x % CB_BLOCKS) * (BLOCK / CELL_LANES) + (int)threadIdx.x / CELL_LANES;
    const int l = threadIdx.x % CELL_LANES;
    double R = 0.0;
    if (c < S.k) {
        const D4 sd = S.seed[c];
        double r2 = 0.0;
        const int b = S.cstart[c], e = b + S.ccount[c];
        for (int i = b + l; i < e; i += CELL_LANES) {
            const D4 p = ld3(S.pos + i);
            double dx, dy, dz;
            r2 = fmax(r2, dist2_exact(S, p.x, p.y, p.z, sd.x, sd.y, sd.z, dx, dy, dz));
        }
        r2 = row_max(r2);
        R = sqrt(r2);
        if (l == CELL_LANES - 1) S.seed[c].w = R;
    }
    if (l != CELL_LANES - 1) R = 0.0;
    for (int o = 32; o > 0; o >>= 1) R = fmax(R, __shfl_xor(R, o));
    if ((threadIdx.x & 63) == 0 && R > 0.0) max_if_larger(&S.sc->rmax, dbits(R));
}

// The query window of cell A on the seed grid: per axis the grid rows within
// R_A + R_max + search of its centroid (a periodic axis wraps; a window that covers
// the period, or a non-finite bound, takes the whole axis).  Along z, whose grid cells
// are consecutive in the grid's linear order, the window is one or two runs of grid
// cells (two where it wraps), so that the seeds of a run are one range of `gseed`.
struct QWin {
    int lo[2], n[2];          // x and y: first row (before wrapping) and row count
    int za[2], zb[2], nz;     // z runs [za, zb] (wrapped), in walk order
};
__device__ __forceinline__ QWin query_window(const SysDev &S, const SysScal *sc, const D4 &ca, double search) {
    const double rho = ca.w + bitsd(sc->rmax) + search + 1e-9;
    const double xa[3] = {ca.x, ca.y, ca.z};
    int lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {
        double u = wrap_coord(xa[a], S.per[a], S.box[a]) - sc->glo[a];
        int dim = sc->gdim[a];
        double fl = floor((u - rho) / sc->gh[a]), fh = floor((u + rho) / sc->gh[a]);
        if (!(fl > -1e9 && fh < 1e9)) { fl = 0.0; fh = (double)(dim - 1); }   // non-finite: scan the axis
        int l = (int)fl;
        int h = (int)fh;
        if (S.per[a]) {
            if (h - l + 1 >= dim) { l = 0; h = dim - 1; }
        } else {
            l = max(l, 0);
            h = min(h, dim - 1);
        }
        lo[a] = l;
        hi[a] = h;
    }
    QWin w;
    for (int a = 0; a < 2; ++a) {
        w.lo[a] = lo[a];
        w.n[a] = max(0, hi[a] - lo[a] + 1);
    }
    const int dz = sc->gdim[2];
    w.nz = 0;
    if (hi[2] >= lo[2]) {
        if (lo[2] < 0) {                  // periodic: the rows below 0 are the top ones, walked first
            w.za[0] = lo[2] + dz; w.zb[0] = dz - 1;
            w.za[1] = 0; w.zb[1] = hi[2];
            w.nz = 2;
        } else if (hi[2] >= dz) {
            w.za[0] = lo[2]; w.zb[0] = dz - 1;
            w.za[1] = 0; w.zb[1] = hi[2] - dz;
            w.nz = 2;
        } else {
            w.za[0] = lo[2]; w.zb[0] = hi[2];
            w.nz = 1;
        }
    }
    return w;
}

// The linear index of grid column (x row, y row) of the window, wrapped on periodic axes.
__device__ __forceinline__ int window_column(const SysDev &S, const SysScal *sc, const QWin &w, int ix, int iy) {
    int gx = w.lo[0] + ix, gy = w.lo[1] + iy;
    if (S.per[0]) gx = ((gx % sc->gdim[0]) + sc->gdim[0]) % sc->gdim[0];
    if (S.per[1]) gy = ((gy % sc->gdim[1]) + sc->gdim[1]) % sc->gdim[1];
    return (gx * sc->gdim[1] + gy) * sc->gdim[2];
}

// Whether seed B pairs with cell A (centroid ca, radius ca.w).
__device__ __forceinline__ bool cell_pair_test(const SysDev &S, const D4 &ca, const D4 &cb, double search) {
    double dx, dy, dz;
    const double d = sqrt(dist2_exact(S, ca.x, ca.y, ca.z, cb.x, cb.y, cb.z, dx, dy, dz));
    return d <= ca.w + cb.w + search + 1e-9;
}

// Cells B paired with A (as below), one thread per cell: the serial walk of the
// window, a column's z runs at a time.  The first cap hits are written, in grid-scan order.
__device__ int cell_query_serial(const SysDev &S, const SysScal *sc, int A, double search, int *out, int cap) {
    const D4 ca = S.seed[A];
    const QWin w = query_window(S, sc, ca, search);
    int cnt = 0;
    for (int ix = 0; ix < w.n[0]; ++ix)
        for (int iy = 0; iy < w.n[1]; ++iy) {
            const int base = window_column(S, sc, w, ix, iy);
            for (int r = 0; r < w.nz; ++r) {
                const int qe = ldg(S.gstart + base + w.zb[r] + 1);
                for (int q = ldg(S.gstart + base + w.za[r]); q < qe; ++q) {
                    const int B = ldg(S.gseed + q);
                    if (cell_pair_test(S, ca, ldg(S.seed + B), search)) {
                        if (cnt < cap) out[cnt] = B;
                        ++cnt;
                    }
                }
            }
        }
    return cnt;
}

// Cells B paired with A: |minimg(c_A - c_B)| <= R_A + R_B + search + 1e-9 with
// search = largest (rc + 2 skin).  One wavefront per cell A: the window's grid columns
// (x slowest) are taken 64 at a time, their seeds laid out in scan order by a scan of their
// counts, and tested 64 at a time, one per lane; the hits are written in that order, the
// first cap of them.  (A lane walking its column's seeds by itself made a chain of two loads
// per seed: 41 us at 6250 cells, now 15.)  Returns the row's length on every lane.
struct QRuns {
    int2 first[WAVE], second[WAVE];                 // a column's runs of seeds: first seed, seeds before the run
    int before[WAVE + 1];                           // candidates before the column
};

__device__ int cell_query_wave(const SysDev &S, const SysScal *sc, int A, double search, QRuns &Q, int32_t *out, int cap) {
    const int lane = threadIdx.x & (WAVE - 1);
    const D4 ca = S.seed[A];
    const QWin w = query_window(S, sc, ca, search);
    const int ncol = w.nz > 0 ? w.n[0] * w.n[1] : 0;
    const double reach = ca.w + bitsd(sc->rmax) + search + 1e-9;
    const bool bounded = reach * reach < INFINITY;
    int total = 0;
    for (int col0 = 0; col0 < ncol; col0 += WAVE) {
        int qb[2] = {0, 0}, n[2] = {0, 0};
        const int col = col0 + lane;
        if (col < ncol) {
            const int base = window_column(S, sc, w, col / w.n[1], col % w.n[1]);
#pragma unroll
            for (int r = 0; r < 2; ++r)
                if (r < w.nz) {
                    qb[r] = ldg(S.gstart + base + w.za[r]);
                    n[r] = ldg(S.gstart + base + w.zb[r] + 1) - qb[r];
                }
        }
        // the candidates of the 64 columns in their order: lane's column starts at `at`
        const int inc = wave_incl_scan(n[0] + n[1]);
        const int at = inc - n[0] - n[1], ncand = __builtin_amdgcn_readlane(inc, WAVE - 1);
        wave_fence();                               // the round before has read its runs
        Q.first[lane] = make_int2(qb[0], 0);
        Q.second[lane] = make_int2(qb[1], n[0]);
        Q.before[lane] = at;
        if (lane == 0) Q.before[WAVE] = ncand;
        wave_fence();
        for (int t0 = 0; t0 < ncand; t0 += WAVE) {
            const int t = t0 + lane;
            int B = -1;
            if (t < ncand) {
                int lo = 0, hi = WAVE;              // the last column that starts at or before t
                while (hi - lo > 1) {
                    const int m = (lo + hi) >> 1;
                    if (Q.before[m] <= t) lo = m;
                    else hi = m;
                }
                const int k = t - Q.before[lo];
                const int2 f = Q.first[lo], g = Q.second[lo];
                const D4 c = ldg(S.gpos + (k < g.y ? f.x + k : g.x + (k - g.y)));
                // the radius is fetched for seeds within the largest one's reach only
                double dx, dy, dz;
                const double d2 = dist2_exact(S, ca.x, ca.y, ca.z, c.x, c.y, c.z, dx, dy, dz);
                if (!bounded || !(d2 > reach * reach * (1.0 + 1e-12))) {
                    const int b = (int)c.w;
                    if (cell_pair_test(S, ca, D4{c.x, c.y, c.z, ldg(&S.seed[b].w)}, search)) B = b;
                }
            }
            const unsigned long long hits = __ballot(B >= 0);
            const int k = total + __popcll(hits & ((1ull << lane) - 1ull));
            if (B >= 0 && k < cap) out[k] = B;
            total += __popcll(hits);
        }
    }
    return total;
}

// Cell-pair kernels.  Systems of at least CQ_SERIAL_MIN cells take one thread per
// cell (there are enough threads to hide the serial walk's latency: 233 us at 225 thousand
// cells, by wavefronts 247); smaller ones give each cell a wavefront (150 thousand: 185 and
// 164 us, 28 thousand: 117 and 42), CQ_BLOCKS blocks per 256-cell block of the cell map.  Both
// find the same rows.
// The query writes a cell's first CROW hits to a scratch row (in the memory of the 32-bit
// fallback lists, idle until the list build) and its row's length; once a scan has placed the
// rows they are copied, and only a longer row (a cell with a far member reaches many) is
// queried again, by a wavefront.  (Querying every cell a
// second time to fill its row took longer than the first time: 41 after 32 us at 6250 cells;
// the copy takes 4 us.)
constexpr int CQ_BLOCKS = BLOCK / (BLOCK / WAVE);
constexpr int CQ_SERIAL_MIN = 200000;
constexpr int CROW = 256;             // (less where cells hold fewer than three particles on average)
__device__ __forceinline__ int crow_of(const SysDev &S) {
    return (int)min((long long)CROW, (long long)S.nchunk * (MAXNB * CHUNK) / S.k);
}
__device__ __forceinline__ int32_t *scratch_row(const SysDev &S, int c) { return S.nl + (size_t)c * crow_of(S); }

// A cell's row length as counted; 0 and an error where it would let the scanned total
// leave int32.
__device__ __forceinline__ int checked_row(const SysDev &S, int c, int n, bool lead) {
    if (n > CNBR_ROW_MAX) {
        if (lead) atomicOr(&S.sc->err, ERR_CNBR);
        n = 0;
    }
    if (lead) S.cnbr_start[c] = n;
    return n;
}

__global__ __launch_bounds__(BLOCK) void k_cnbr_query_serial(const SysDev *Sd, Maps L_maps, double search) {
    SYS_FROM(c);
    if (!S.sc->rebuild || S.k < CQ_SERIAL_MIN) return;
    const int c = lb * BLOCK + threadIdx.x;
    int n = 0;
    if (c < S.k) n = checked_row(S, c, cell_query_serial(S, S.sc, c, search, scratch_row(S, c), crow_of(S)), true);
    const int m = wave_max_int(n);
    if ((threadIdx.x & 63) == 0 && m > 0) max_if_larger(&S.sc->cnbr_maxrow, m);
}

__global__ __launch_bounds__(BLOCK) void k_cnbr_query(const SysDev *Sd, Maps L_maps, double search) {
    const int cbk = blockIdx.x / CQ_BLOCKS;
    if (cbk >= L_maps.c[L_maps.nsys]) return;
    const int s = find_sys(L_maps.c, L_maps.nsys, cbk);
    const SysDev &S = Sd[s];
    if (!S.sc->rebuild || S.k >= CQ_SERIAL_MIN) return;
    const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
    const int c = (cbk - L_maps.c[s]) * BLOCK + (blockIdx.x % CQ_BLOCKS) * (BLOCK / WAVE) + wv;
    __shared__ QRuns s_q[BLOCK / WAVE];
    int m = 0;
    if (c < S.k)                                   // wavefront-uniform
        m = checked_row(S, c, cell_query_wave(S, S.sc, c, search, s_q[wv], scratch_row(S, c), crow_of(S)), lane == 0);
    __shared__ int s_m[BLOCK / WAVE];
    if (lane == 0) s_m[wv] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int mm = max(max(s_m[0], s_m[1]), max(s_m[2], s_m[3]));
        if (mm > 0) max_if_larger(&S.sc->cnbr_maxrow, mm);
    }
}

// The rows to their places, CELL_LANES lanes per cell.
__global__ __launch_bounds__(BLOCK) void k_cnbr_place(const SysDev *Sd, Maps L_maps, double search) {
    const int cbk = blockIdx.x / CB_BLOCKS;
    const int s = find_sys(L_maps.c, L_maps.nsys, cbk);
    const SysDev &S = Sd[s];
    if (!S.sc->rebuild) return;
    const int c = (cbk - L_maps.c[s]) * BLOCK + (blockIdx.x % CB_BLOCKS) * (BLOCK / CELL_LANES) + (int)threadIdx.x / CELL_LANES;
    const int l = threadIdx.x % CELL_LANES;
    const bool lead = c == 0 && l == 0;
    const int total = S.cnbr_start[S.k];
    if (lead) S.sc->cnbr_total = total;
    if (total > S.cnbr_cap || (S.sc->err & ERR_CNBR)) {
        if (lead) atomicOr(&S.sc->err, ERR_CNBR);
        return;
    }
    __shared__ QRuns s_q[BLOCK / WAVE];
    __shared__ int s_long[CPB];
    const int cap = crow_of(S), g = threadIdx.x / CELL_LANES;
    const int b = c < S.k ? S.cnbr_start[c] : 0, n = c < S.k ? S.cnbr_start[c + 1] - b : 0;
    if (l == 0) s_long[g] = n > cap ? n : 0;
    if (n <= cap && n > 0) {
        const int32_t *row = scratch_row(S, c);
        for (int q = l; q < n; q += CELL_LANES) S.cnbr[b + q] = row[q];
    }
    __syncthreads();
    for (int h = threadIdx.x / WAVE; h < CPB; h += BLOCK / WAVE)           // wavefront-uniform
        if (s_long[h]) {
            const int cl = c - g + h;
            (void)cell_query_wave(S, S.sc, cl, search, s_q[threadIdx.x / WAVE], S.cnbr + S.cnbr_start[cl], s_long[h]);
        }
}

void launch_cell_bounds(const LaunchCtx &L) {
    hipLaunchKernelGGL(k_cell_bounds, dim3(CB_BLOCKS * L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps);
}

void launch_cell_pairs(const LaunchCtx &L) {
    if (L.nblk_c == 0) return;
    // each size class's query only where the launch holds a system of that class
    if (L.kmax >= CQ_SERIAL_MIN)
        hipLaunchKernelGGL(k_cnbr_query_serial, dim3(L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps, L.prm.cell_search);
    if (L.kmin < CQ_SERIAL_MIN)
        hipLaunchKernelGGL(k_cnbr_query, dim3(CQ_BLOCKS * L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps,
                           L.prm.cell_search);
    launch_scan(L, 3);
    hipLaunchKernelGGL(k_cnbr_place, dim3(CB_BLOCKS * L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps, L.prm.cell_search);
}

// ------------------------------------------------------------------ neighbour lists

__device__ __forceinline__ int lds_lower_bound(const int *a, int n, int v) {
    int lo = 0, hi = n;
    while (lo < hi) {
        int m = (lo + hi) >> 1;
        if (a[m] < v) lo = m + 1; else hi = m;
    }
    return lo;
}

// One of three FP32 radii by partner type, as integer selects (no branches).
__device__ __forceinline__ float sel3f(int t, float a, float b, float c) {
    int r = (t == 1) ? __float_as_int(b) : __float_as_int(c);
    r = (t == 0) ? __float_as_int(a) : r;
    return __int_as_float(r);
}

// A block's stage entries in LDS: FP32 offsets from the block's first particle, and a byte
// with the type and, once a pruned list uses the entry, STAGE_USED.  The used entries are
// marked with plain byte stores: many lanes' atomics on a few bitmap words would serialise.
constexpr unsigned char STAGE_USED = 4;

// The USED bits of 32 such bytes (4-byte aligned) as one word, entry k in bit k.
__device__ __forceinline__ unsigned pack_used(const unsigned char *f) {
    const unsigned *w = reinterpret_cast<const unsigned *>(f);
    unsigned bits = 0u;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const unsigned v = w[q] >> 2;
        bits |= ((v & 1u) | ((v >> 7) & 2u) | ((v >> 14) & 4u) | ((v >> 21) & 8u)) << (4 * q);
    }
    return bits;
}

// The pruned stage of a block: the used ones of its scnt stage entries, in stage order
// (entries to istage), and for every 32 entries their bits and rank in bp.  Returns its size.
__device__ int pruned_stage(const SysDev &S, int lb, int scnt, const unsigned char *s_tf, uint2 *s_bp, int *s_w) {
    const int nwords = (scnt + 31) / 32;                 // at most SMAX / 32 = 64: one wavefront's
    static_assert(SMAX / 32 <= WAVE, "the words of a stage");
    __syncthreads();
    if (threadIdx.x < WAVE) {
        const int w = threadIdx.x;
        const unsigned bits = w < nwords ? pack_used(s_tf + 32 * w) : 0u;
        const int c = __popc(bits);
        const int x = wave_incl_scan(c);
        s_bp[w] = make_uint2(bits, (unsigned)(x - c));
        if (w == WAVE - 1) s_w[0] = x;
    }
    __syncthreads();
    for (int k = threadIdx.x; k < scnt; k += BLOCK) {
        const uint2 b = s_bp[k >> 5];
        const unsigned m = 1u << (k & 31);
        if (b.x & m)
            stg(S.istage + (size_t)lb * SSTRIDE + b.y + __popc(b.x & (m - 1u)), ldg(S.stage + (size_t)lb * SSTRIDE + k));
    }
    return s_w[0];
}

// The pruned lists of a wavefront's chunk from its full lists (`rows` rows) and the bits
// of the rows that stay (pm): each lane's entries become indices into the pruned stage,
// are gathered in its own dwords of an LDS buffer (PAIRS row pairs; entries beyond it go
// straight to memory) and leave as whole row pairs, padded with 0xffff to the chunk's row
// count rounded up to even (the step kernel takes rows in pairs).
template <int PAIRS>
__device__ void emit_pruned(const SysDev &S, int chunk, int rows, unsigned pm0, unsigned pm1, unsigned pm2,
                            const uint2 *s_bp, uint16_t *s_buf) {
    const int tid = threadIdx.x, lane = tid & (WAVE - 1);
    const int mine = __popc(pm0) + __popc(pm1) + __popc(pm2);
    const int irows = wave_max_int(mine);
    if (lane == 0) S.ilk[chunk] = irows;
    const v4u *src = reinterpret_cast<const v4u *>(S.nl16 + (size_t)chunk * MAXNB * CHUNK) + lane;
    uint16_t *dst = S.il16 + (size_t)chunk * MAXNB * CHUNK;
    const int ng = (rows + 7) / 8;
    int pc = 0;
    v4u nxt = {0u, 0u, 0u, 0u};
    if (ng > 0) nxt = ldg(src);
    for (int g = 0; g < ng; ++g) {
        const v4u e = nxt;
        if (g + 1 < ng) nxt = ldg(src + (g + 1) * CHUNK);
        const unsigned pb = (g < 4 ? pm0 : (g < 8 ? pm1 : pm2)) >> (8 * (g & 3));
        unsigned local[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {                // the eight ranks side by side
            unsigned k = (q & 1) ? e[q >> 1] >> 16 : e[q >> 1] & 0xffffu;
            k = (pb >> q) & 1u ? k : 0u;
            const uint2 b = s_bp[k >> 5];
            local[q] = il_entry(b.y + __popc(b.x & ((1u << (k & 31)) - 1u)));
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if ((pb >> q) & 1u) {
                if (pc < 2 * PAIRS) s_buf[(pc >> 1) * (2 * BLOCK) + 2 * tid + (pc & 1)] = (uint16_t)local[q];
                else stg(dst + il_at(pc, lane), (uint16_t)local[q]);
                ++pc;
            }
        }
    }
    const unsigned *s_b32 = reinterpret_cast<const unsigned *>(s_buf);
    for (int p = 0, np = (irows + 1) >> 1; p < np; ++p) {
        const int r = 2 * p;
        if (p < PAIRS) {
            unsigned v = s_b32[p * BLOCK + tid];
            v = r + 1 < mine ? v : (r < mine ? v | 0xffff0000u : 0xffffffffu);
            stg(reinterpret_cast<unsigned *>(dst + il_at(r, lane)), v);
        } else {
            if (r >= mine) stg(dst + il_at(r, lane), (uint16_t)0xffff);
            if (r + 1 >= mine) stg(dst + il_at(r + 1, lane), (uint16_t)0xffff);
        }
    }
}

// Last candidate cell whose particle offset is <= u (offsets of empty cells repeat).
__device__ __forceinline__ int union_cell(const int *ofs, int nsc, int u) {
    int lo = 0, hi = nsc;
    while (hi - lo > 1) {
        const int m = (lo + hi) >> 1;
        if (ofs[m] <= u) lo = m; else hi = m;
    }
    return lo;
}

// One block per 256 consecutive cell-sorted particles (four 64-particle chunks), whose
// cells are consecutive: the block's own cells.
//  - Candidate cells: the cell-pair entries of the own cells, sorted and deduplicated in
//    LDS (the union).
//  - Stage: the union's particles that lie within the list radius of some own cell's
//    bounding sphere, of those own cells that pair with the particle's cell (a 64-bit
//    mask per union cell), in the union's order, as FP32 offsets from the block's first
//    particle.  A superset of the block's partners.  Each entry keeps a bit for every own
//    cell whose sphere test it passed.  A wide cell (one with a member far off) would pass
//    thousands of particles that are near none of its members: it is tested as one small
//    sphere per member instead, where the block's spheres still fit 64 in all.  (One such
//    cell had left its block of a deformed 125k-particle vesicle without a stage: 6.4 ms
//    instead of 1.5 ms per 20 steps.)  Blocks of more than 64 own cells take runs of them as
//    one sphere each.  Where large cells, of which the block holds a part, pass more than the
//    stage holds, a second pass keeps only what is also near the boxes of the block's chunks
//    (1M particles in cells of 1000: 24% of the blocks staged and 14.8 ms without it, 81% and
//    7.5 ms with it).
//  - Candidate lists: for each own cell the stage entries with its bit, compacted by one
//    wavefront's ballots as 16-bit LDS offsets, lipids from the front, proteins from the
//    back (neighbouring cells share a list where a block has more than 16).  Every
//    particle of a cell scans the same short list (about 130 entries for 47 partners at
//    skin 0.65), so that the wavefront's lanes run through it together, each segment with
//    one radius.  As many lists are built at a time as fit the buffer; nearly always that
//    is all of them.
//  - Scan: each lane tests its cell's candidates against the list radius (rc + 2 skin of
//    the pair's types) and keeps a bit for each, in words in LDS.  The test runs in FP32
//    against the radius widened by 1e-3 sigma, which bounds the offsets' rounding (offsets
//    are limited to 4096 sigma), so the list is a superset of the FP64 one; the step
//    kernel decides every pair exactly.
//  - Lists: the lanes take their next set bit row by row together, eight rows to a
//    16-byte store.  The same pass tests the pruned radius (rc + 2 inner skin), marks the
//    stage entries that pass and keeps a bit per row; emit_pruned then writes the pruned
//    lists.  Hits beyond the words that fit are appended one by one.  A lane with more than
//    MAXNB hits starts again at a shorter radius (NL_LEVELS).
// What bounds it is latency: three blocks of four wavefronts share a CU, and every phase is
// a chain of loads, barriers and LDS reads, so each is written with as many of them side
// by side as it has (four union particles, eight candidates, eight rows at a time).
// Blocks whose stage does not fit, or with more than CANDMAX cell pairs, keep 32-bit lists of
// global slots (stage count -1), built on FP64 positions by a slow serial scan.
constexpr int UCELLS = CANDMAX;       // candidate (union) cells per block
constexpr int OWNMAX = 64;            // spheres of a block's own cells
constexpr int GROUPS = 16;            // candidate lists of a block
constexpr int CLIST = 5120;           // candidate-list entries of those cells
constexpr int MWORDS = 11;            // words of hit bits per lane (352 candidates)
// A cell is wide from this many list radii on: its sphere covers (1 + 1.5)^2 = 6 times the
// area in which one of its members can have partners; compact cells have 0.5 to 1.
constexpr float WIDE = 1.5f;

__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(1, 3))) void k_nlist(const SysDev *Sd, Maps L_maps, DevParams P) {
    SYS_FROM(p);
    if (!S.sc->rebuild) return;
    // 53 KB of LDS, three blocks per CU.  s_raw: the stage's x, y, z; the union arrays, then
    // the candidate lists; the own particles' stage entries, then the hit words; before the
    // stage, the union's sort; after the scan, the pruned stage's words and the row buffer.
    constexpr int RX = 3 * USTAGE * 4, RL = 2 * CLIST, RM = MWORDS * BLOCK * 4;
    __shared__ __align__(16) unsigned char s_raw[RX + RL + RM];
    __shared__ __align__(16) unsigned char s_tf[USTAGE];    // type | STAGE_USED of the stage entries
    __shared__ uint16_t s_q[USTAGE];                        // union position of every cell-pair entry; then the
                                                            // stage entries' own-list bits
    __shared__ F4 s_sph[OWNMAX];                            // spheres of the own cells: offset and widened radius
    __shared__ uint16_t s_ibeg[OWNMAX];                     // the first sphere of an own cell (or run) and their number
    __shared__ float s_box[BLOCK / WAVE][6];                // boxes of the chunks: centre, half width
    __shared__ int s_lofs[GROUPS + 1];
    __shared__ uint16_t s_nl[GROUPS], s_np[GROUPS];         // lipid and protein candidates of each list
    __shared__ int s_w[16];
    __shared__ int s_rows[BLOCK / WAVE], s_big, s_nfit;
    uint16_t *s_qpos = s_q, *s_om = s_q;
    static_assert(CANDMAX <= USTAGE && GROUPS <= 16, "list bits");
    float *s_ux = reinterpret_cast<float *>(s_raw), *s_uy = s_ux + USTAGE, *s_uz = s_uy + USTAGE;
    int *s_cand = reinterpret_cast<int *>(s_raw + RX);
    int *s_ofs = s_cand + UCELLS;
    unsigned long long *s_mask = reinterpret_cast<unsigned long long *>(s_ofs + UCELLS + 2);
    uint16_t *s_list = reinterpret_cast<uint16_t *>(s_raw + RX);
    uint16_t *s_self = reinterpret_cast<uint16_t *>(s_raw + RX + RL + RM) - BLOCK;
    static_assert(RL + RM - 2 * BLOCK >= (2 * UCELLS + 2) * (int)sizeof(int) + UCELLS * (int)sizeof(unsigned long long), "union arrays");
    unsigned *s_m = reinterpret_cast<unsigned *>(s_raw + RX + RL);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int chunk = lb * (BLOCK / WAVE) + wv;
    const bool chunk_ok = chunk < S.nchunk;
    const int i = lb * BLOCK + tid;
    const bool valid = i < S.n;
    const int first = lb * BLOCK;
    const D4 ref = ld3(S.pos + first);
    const D4 pi = valid ? ldpos(S, i) : ref;
    if (valid) {
        // the drift references of the new lists
        const F3 b = {(float)pi.x, (float)pi.y, (float)pi.z};
        S.xb[i] = b;
        S.xp[i] = b;
    }
    if (S.sc->err & ERR_CNBR) {          // no valid cell pairs: publish empty lists (block-uniform)
        if (lane == 0 && chunk_ok) { S.nlk[chunk] = 0; S.ilk[chunk] = 0; }
        if (tid == 0) { S.scount[lb] = 0; S.iscount[lb] = 0; }
        return;
    }
    if (tid == 0) s_big = 0;             // raised after the union's barriers
    reinterpret_cast<uint2 *>(s_tf)[tid] = make_uint2(0u, 0u);
    static_assert(USTAGE == 8 * BLOCK, "type bytes");
    // ---- candidate cells and the union position of every cell-pair entry
    const int last = min(S.n - 1, first + BLOCK - 1);
    const int c0 = S.owner[first], c1 = S.owner[last];
    const int A = valid ? ldg(S.owner + i) : c0;
    const int q0 = S.cnbr_start[c0];
    const int ncand = S.cnbr_start[c1 + 1] - q0;
    const int nown = c1 - c0 + 1;
    const bool have_union = !(ncand <= 0 || ncand > CANDMAX || c1 < c0);
    // own cells to a sphere, 1 << rs (a cell pairs with itself: nown is at most CANDMAX)
    int rs = 0;
    while (have_union && (nown - 1) >> rs >= OWNMAX) ++rs;
    const int nsph = ((nown - 1) >> rs) + 1;
    const bool periodic = (S.per[0] | S.per[1] | S.per[2]) != 0;
    const float Lx = S.per[0] ? (float)S.box[0] : 0.0f, Ly = S.per[1] ? (float)S.box[1] : 0.0f,
                Lz = S.per[2] ? (float)S.box[2] : 0.0f;
    const float iLx = S.per[0] ? 1.0f / Lx : 0.0f, iLy = S.per[1] ? 1.0f / Ly : 0.0f, iLz = S.per[2] ? 1.0f / Lz : 0.0f;
    const double iL[3] = {S.per[0] ? 1.0 / S.box[0] : 0.0, S.per[1] ? 1.0 / S.box[1] : 0.0, S.per[2] ? 1.0 / S.box[2] : 0.0};
    // FP32 offset from the block's first particle (any image: the tests take the nearest)
    auto offset = [&](int a, double x, double x0) {
        const double d = x - x0;
        return (float)(periodic && S.per[a] ? minimg_fast(d, S.box[a], iL[a]) : d);
    };
    int nsc = 0, ss = 0;
    if (have_union) {
        // the range of the candidate cell ids: where it spans at most CANDBITS ids, a
        // bitmap over it and the words' prefix counts sort and deduplicate them; otherwise
        // a bitonic sort does (both in the stage's memory)
        int *s_srt = reinterpret_cast<int *>(s_raw);
        int cv[CANDMAX / BLOCK];         // this thread's entries
        int mn = INT_MAX, mx = INT_MIN;
#pragma unroll
        for (int k = 0; k < CANDMAX / BLOCK; ++k) {
            const int q = tid + k * BLOCK;
            cv[k] = q < ncand ? ldg(S.cnbr + q0 + q) : -1;
        }
#pragma unroll
        for (int k = 0; k < CANDMAX / BLOCK; ++k)
            if (cv[k] >= 0) {
                mn = min(mn, cv[k]);
                mx = max(mx, cv[k]);
            }
        for (int o = 32; o > 0; o >>= 1) {
            mn = min(mn, __shfl_xor(mn, o));
            mx = max(mx, __shfl_xor(mx, o));
        }
        if (lane == 0) { s_w[wv] = mn; s_w[8 + wv] = mx; }
        __syncthreads();
        mn = min(min(s_w[0], s_w[1]), min(s_w[2], s_w[3]));
        mx = max(max(s_w[8], s_w[9]), max(s_w[10], s_w[11]));
        __syncthreads();
        if (mx - mn < CANDBITS) {
            unsigned *bm = reinterpret_cast<unsigned *>(s_srt);
            int *wpre = s_srt + CANDBITS / 32;
            static_assert(3 * USTAGE * sizeof(float) >= 2 * (CANDBITS / 32) * sizeof(int), "the bitmap");
            const int nw = ((mx - mn) >> 5) + 1;
            for (int w = tid; w < nw; w += BLOCK) bm[w] = 0u;
            __syncthreads();
#pragma unroll
            for (int k = 0; k < CANDMAX / BLOCK; ++k)
                if (cv[k] >= 0) atomicOr(&bm[(cv[k] - mn) >> 5], 1u << ((cv[k] - mn) & 31));
            __syncthreads();
            // prefix counts of the words, a run of consecutive words per thread
            const int per = (nw + BLOCK - 1) / BLOCK, w0 = tid * per, w1 = min(nw, w0 + per);
            int cnt = 0;
            for (int w = w0; w < w1; ++w) cnt += __popc(bm[w]);
            int r = block_excl_scan(cnt, s_w, nsc);
            for (int w = w0; w < w1; ++w) {
                unsigned b = bm[w];
                wpre[w] = r;
                while (b) {
                    s_cand[r++] = mn + (w << 5) + (__ffs(b) - 1);
                    b &= b - 1u;
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < CANDMAX / BLOCK; ++k)
                if (cv[k] >= 0) {
                    const int v = cv[k] - mn;
                    s_qpos[tid + k * BLOCK] = (uint16_t)(wpre[v >> 5] + __popc(bm[v >> 5] & ((1u << (v & 31)) - 1u)));
                }
        } else {
            int pw = 1;
            while (pw < ncand) pw <<= 1;
#pragma unroll
            for (int k = 0; k < CANDMAX / BLOCK; ++k) s_srt[tid + k * BLOCK] = cv[k] >= 0 ? cv[k] : INT_MAX;
            __syncthreads();
            for (int kk = 2; kk <= pw; kk <<= 1)
                for (int jj = kk >> 1; jj > 0; jj >>= 1) {
                    for (int t = tid; t < pw; t += BLOCK) {
                        int ixj = t ^ jj;
                        if (ixj > t) {
                            int va = s_srt[t], vb = s_srt[ixj];
                            bool up = (t & kk) == 0;
                            if ((va > vb) == up) { s_srt[t] = vb; s_srt[ixj] = va; }
                        }
                    }
                    __syncthreads();
                }
            // deduplicate into the union
            int vals[CANDMAX / BLOCK], fl[CANDMAX / BLOCK], loc = 0;
            for (int q = 0; q < CANDMAX / BLOCK; ++q) {
                const int idx = tid * (CANDMAX / BLOCK) + q;
                vals[q] = idx < pw ? s_srt[idx] : INT_MAX;
                const int prev = (idx > 0 && idx < pw) ? s_srt[idx - 1] : INT_MIN;
                fl[q] = (idx < ncand && (idx == 0 || vals[q] != prev)) ? 1 : 0;
                loc += fl[q];
            }
            int p = block_excl_scan(loc, s_w, nsc);
            for (int q = 0; q < CANDMAX / BLOCK; ++q)
                if (fl[q]) s_cand[p++] = vals[q];
            __syncthreads();
#pragma unroll
            for (int k = 0; k < CANDMAX / BLOCK; ++k)
                if (cv[k] >= 0) s_qpos[tid + k * BLOCK] = (uint16_t)lds_lower_bound(s_cand, nsc, cv[k]);
        }
        __syncthreads();
    }
    // ---- the stage
    float oi[3] = {offset(0, pi.x, ref.x), offset(1, pi.y, ref.y), offset(2, pi.z, ref.z)};
    if (!valid) oi[0] = oi[1] = oi[2] = 0.0f;
    // offsets beyond LIST_EXTENT (or not finite) leave the block without a stage
    auto far = [](const float o[3]) {
        return !(fabsf(o[0]) <= LIST_EXTENT && fabsf(o[1]) <= LIST_EXTENT && fabsf(o[2]) <= LIST_EXTENT);
    };
    auto dist2f = [&](float ax, float ay, float az, float x, float y, float z) {
        float dx = ax - x, dy = ay - y, dz = az - z;
        if (periodic) {
            dx -= Lx * rintf(dx * iLx);
            dy -= Ly * rintf(dy * iLy);
            dz -= Lz * rintf(dz * iLz);
        }
        return dx * dx + dy * dy + dz * dz;
    };
    // the bounding sphere of own cell a (radius widened by 2e-3 sigma for the offsets' rounding)
    auto own_sphere = [&](int a) {
        const D4 c = ldg(S.seed + c0 + a);
        const float o[3] = {offset(0, c.x, ref.x), offset(1, c.y, ref.y), offset(2, c.z, ref.z)};
        if (far(o)) s_big = 1;
        return F4{o[0], o[1], o[2], (float)c.w + 2e-3f};
    };
    // a sphere with its candidate list's number in the radius' last bits (rounded up)
    auto tagged = [](F4 s, int g) {
        static_assert(GROUPS == 16, "four bits");
        s.w = __int_as_float(((__float_as_int(s.w) + 16) & ~15) | g);
        return s;
    };
    // candidate list of sphere a's own cells
    auto group_of = [&](int a) { return nsph <= GROUPS ? a : a * GROUPS / nsph; };
    // one sphere about own cells [a, e): centred on the middle one, round all that hold particles
    auto run_sphere = [&](int a, int e) {
        const D4 m = ldg(S.seed + c0 + ((a + e) >> 1));
        double r = 0.0;
        for (int c = a; c < e; ++c)
            if (ldg(S.ccount + c0 + c) > 0) {
                const D4 q = ldg(S.seed + c0 + c);
                double dx, dy, dz;
                r = fmax(r, q.w + sqrt(dist2_exact(S, m.x, m.y, m.z, q.x, q.y, q.z, dx, dy, dz)));
            }
        const float o[3] = {offset(0, m.x, ref.x), offset(1, m.y, ref.y), offset(2, m.z, ref.z)};
        if (far(o)) s_big = 1;
        return F4{o[0], o[1], o[2], (float)r + 2e-3f};
    };
    // list radius of a candidate by its type (the largest over the own types)
    const float rlm0 = P.rlmaxf[0], rlm1 = P.rlmaxf[1], rlm2 = P.rlmaxf[2];
    int kept = 0;
    if (have_union) {
        constexpr int PER = UCELLS / BLOCK;
        static_assert(UCELLS == PER * BLOCK, "cells per thread");
        int ccnt[PER], loc = 0;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int c = tid * PER + q;
            ccnt[q] = c < nsc ? ldg(S.ccount + s_cand[c]) : 0;
            loc += ccnt[q];
            if (c < nsc) s_mask[c] = 0ull;
        }
        if (wv == 0) {
            // own cell `lane`: its first sphere, the number beyond one, and whether they are
            // its members'
            F4 sp = {0.0f, 0.0f, 0.0f, 0.0f};
            int m = 0;
            if (lane < nsph) {
                sp = rs == 0 ? own_sphere(lane) : run_sphere(lane << rs, min(nown, (lane + 1) << rs));
                if (rs == 0 && sp.w > WIDE * fmaxf(fmaxf(rlm0, rlm1), rlm2)) {
                    const int b = ldg(S.cstart + c0 + lane), e = b + ldg(S.ccount + c0 + lane);
                    m = max(min(e, last + 1) - max(b, first), 0);
                }
            }
            const int room = wave_incl_scan(max(m - 1, 0));
            const bool wide = m > 0 && room <= OWNMAX - nsph;
            const int more = wide ? m - 1 : 0;
            const int at = wave_incl_scan(more) - more + lane;
            if (lane < nsph) {
                s_ibeg[lane] = (uint16_t)(at | (more << 8) | (wide ? 0x8000 : 0));
                if (!wide) s_sph[at] = tagged(sp, group_of(lane));
            }
        }
        int ex = block_excl_scan(loc, s_w, ss);
        if (valid) {
            const int v = s_ibeg[(A - c0) >> rs];
            if (v & 0x8000)
                s_sph[(v & 255) + i - max(ldg(S.cstart + A), first)] = tagged(F4{oi[0], oi[1], oi[2], 2e-3f}, group_of(A - c0));
        }
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int c = tid * PER + q;
            if (c <= nsc) s_ofs[c] = ex;
            ex += ccnt[q];
        }
        if (tid == 0 && nsc == UCELLS) s_ofs[nsc] = ss;
        for (int a = wv; a < nown; a += BLOCK / WAVE) {
            const int b = ldg(S.cnbr_start + c0 + a) - q0, e = ldg(S.cnbr_start + c0 + a + 1) - q0;
            const int v = s_ibeg[a >> rs];
            const unsigned long long bits = (~0ull >> (63 - ((v >> 8) & 127))) << (v & 255);
            for (int q = b + lane; q < e; q += WAVE) atomicOr(&s_mask[s_qpos[q]], bits);
        }
        __syncthreads();
        constexpr int SB = 4;                       // union particles per thread in flight
        // whether an offset lies within the largest list radius of a chunk's box (a periodic axis
        // of which the box spans a quarter or more counts as within)
        const float rb = fmaxf(rlm0, fmaxf(rlm1, rlm2)) + 1e-3f;
        auto near_boxes = [&](const float (&q)[3]) __attribute__((always_inline)) {
            float best = INFINITY;
#pragma unroll 1
            for (int w = 0; w < BLOCK / WAVE; ++w) {
                float e2 = 0.0f;
#pragma unroll
                for (int a = 0; a < 3; ++a) {
                    const float L = a == 0 ? Lx : (a == 1 ? Ly : Lz), iL1 = a == 0 ? iLx : (a == 1 ? iLy : iLz);
                    float d = q[a] - s_box[w][a];
                    if (periodic) d -= L * rintf(d * iL1);
                    const float e = fmaxf(fabsf(d) - s_box[w][3 + a], 0.0f);
                    e2 += e * e;
                }
                best = fminf(best, e2);
            }
            return best <= rb * rb;
        };
        for (bool boxes = false;; boxes = true) {
            kept = 0;
            for (int u0 = 0; u0 < ss; u0 += SB * BLOCK) {
                int c[SB], slot[SB];
                float o[SB][3], rm[SB];
                int t[SB];
                D4 pj[SB];
                unsigned lo[SB], hi[SB], om[SB], any = 0u, anyhi = 0u;
#pragma unroll
                for (int k = 0; k < SB; ++k) {
                    const int u = u0 + k * BLOCK + tid;
                    c[k] = u < ss ? union_cell(s_ofs, nsc + 1, u) : -1;
                    slot[k] = c[k] >= 0 ? ldg(S.cstart + s_cand[c[k]]) + (u - s_ofs[c[k]]) : first;
                }
#pragma unroll
                for (int k = 0; k < SB; ++k) pj[k] = ldpos(S, slot[k]);
#pragma unroll
                for (int k = 0; k < SB; ++k) {
                    o[k][0] = offset(0, pj[k].x, ref.x);
                    o[k][1] = offset(1, pj[k].y, ref.y);
                    o[k][2] = offset(2, pj[k].z, ref.z);
                    if (c[k] >= 0 && far(o[k])) s_big = 1;
                    t[k] = (int)pj[k].w & 3;
                    rm[k] = sel3f(t[k], rlm0, rlm1, rlm2);
                    const unsigned long long m = c[k] >= 0 ? s_mask[c[k]] : 0ull;
                    lo[k] = (unsigned)m;
                    hi[k] = (unsigned)(m >> 32);
                    om[k] = 0u;
                    any |= lo[k];
                    anyhi |= hi[k];
                }
                // the own cells' spheres, the four particles' next ones side by side
                auto spheres = [&](unsigned (&m)[SB], unsigned more, int base) {
                    while (more) {
                        more = 0u;
#pragma unroll
                        for (int k = 0; k < SB; ++k) {
                            const int a = base + (m[k] ? __ffs(m[k]) - 1 : 0);
                            const F4 sp = s_sph[a];
                            const float rr = sp.w + rm[k];
                            if (m[k] && dist2f(sp.x, sp.y, sp.z, o[k][0], o[k][1], o[k][2]) <= rr * rr)
                                om[k] |= 1u << (__float_as_int(sp.w) & 15);
                            m[k] &= m[k] - 1u;
                            more |= m[k];
                        }
                    }
                };
                spheres(lo, any, 0);
                spheres(hi, anyhi, 32);
                if (boxes) {
#pragma unroll
                    for (int k = 0; k < SB; ++k)
                        if (!near_boxes(o[k])) om[k] = 0u;
                }
                // places: by round, wavefront and lane (the union's order)
                int rank[SB];
#pragma unroll
                for (int k = 0; k < SB; ++k) {
                    const unsigned long long b = __ballot(om[k] != 0u);
                    rank[k] = __popcll(b & ((1ull << lane) - 1ull));
                    if (lane == 0) s_w[k * (BLOCK / WAVE) + wv] = __popcll(b);
                }
                static_assert(SB * (BLOCK / WAVE) == 16, "counts of a pass");
                __syncthreads();
                int run = kept;
#pragma unroll
                for (int k = 0; k < SB; ++k) {
#pragma unroll
                    for (int w = 0; w < BLOCK / WAVE; ++w) {
                        if (w == wv) rank[k] += run;
                        run += s_w[k * (BLOCK / WAVE) + w];
                    }
                    if (om[k] && rank[k] < USTAGE) {
                        s_ux[rank[k]] = o[k][0];
                        s_uy[rank[k]] = o[k][1];
                        s_uz[rank[k]] = o[k][2];
                        s_tf[rank[k]] = (unsigned char)t[k];
                        s_om[rank[k]] = (uint16_t)om[k];
                        stg(S.stage + (size_t)lb * SSTRIDE + rank[k], stage_entry(slot[k], t[k]));
                        if ((unsigned)(slot[k] - first) < (unsigned)BLOCK) s_self[slot[k] - first] = (uint16_t)rank[k];
                    }
                }
                kept = run;                              // (beyond USTAGE: no stage)
                __syncthreads();
            }
            // the chunks' boxes, and the stage once more, where the own cells have at least as many
            // members outside the block (a block that holds its cells whole gains nothing: 20
            // thousand vesicle particles with protein cells, an update 544 us, 612 with it)
            if (kept <= USTAGE || boxes) break;     // block-uniform, as is what follows
            if (ldg(S.cstart + c1) + ldg(S.ccount + c1) - ldg(S.cstart + c0) < 2 * BLOCK) break;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                float mn = valid ? oi[a] : INFINITY, mx = valid ? oi[a] : -INFINITY;
                for (int x = 32; x > 0; x >>= 1) {
                    mn = fminf(mn, __shfl_xor(mn, x));
                    mx = fmaxf(mx, __shfl_xor(mx, x));
                }
                const float L = a == 0 ? Lx : (a == 1 ? Ly : Lz), half = 0.5f * (mx - mn) + 1e-3f;
                if (lane == 0) {
                    s_box[wv][a] = mn <= mx ? 0.5f * (mn + mx) : 0.0f;
                    s_box[wv][3 + a] = !(mn <= mx) ? -INFINITY : (L > 0.0f && !(4.0f * (half + rb) < L) ? INFINITY : half);
                }
            }
            __syncthreads();
        }
    }
    const bool staged = have_union && kept <= USTAGE && s_big == 0;
    // ---- the lists, and the bits of the rows that the pruned lists keep
    int cnt = 0, mygroups = 0, level = 0;            // this lane's partners, groups of eight rows written, radius
    unsigned pm0 = 0u, pm1 = 0u, pm2 = 0u;
    static_assert(MAXNB == 96, "row bits in three words");
    const int ti = (int)pi.w & 3;
    uint16_t *row = S.nl16 + (size_t)(chunk_ok ? chunk : 0) * MAXNB * CHUNK;
    v4u *row8 = reinterpret_cast<v4u *>(row) + lane;
    if (staged) {
        const float oix = oi[0], oiy = oi[1], oiz = oi[2];
        const float rlA = P.rl2f[ti][0], rlB = P.rl2f[ti][1], rlC = P.rl2f[ti][2];
        const float riA = P.rin2f[ti][0], riB = P.rin2f[ti][1], riC = P.rin2f[ti][2];
        const int oself = valid ? 4 * (int)s_self[tid] : -1;     // this particle's own stage entry (LDS offset)
        const int G = min(nsph, GROUPS), mygrp = group_of((A - c0) >> rs);
        auto ux = [&](int o) { return *reinterpret_cast<const float *>(s_raw + o); };
        auto uy = [&](int o) { return *reinterpret_cast<const float *>(s_raw + 4 * USTAGE + o); };
        auto uz = [&](int o) { return *reinterpret_cast<const float *>(s_raw + 8 * USTAGE + o); };
        // one entry (LDS offset o, type t) as row r of this lane, with its bit of the pruned rows
        auto append = [&](int r, int o, int t, bool in) __attribute__((always_inline)) {
            if ((r & 7) == 0) {
                stg(row8 + (r >> 3) * CHUNK, v4u{~0u, ~0u, ~0u, ~0u});
                mygroups = (r >> 3) + 1;
            }
            stg(row + nl_at(r, lane), (uint16_t)(o >> 2));
            if (in) {
                const unsigned bit = 1u << (r & 31);
                if (r < 32) pm0 |= bit;
                else if (r < 64) pm1 |= bit;
                else pm2 |= bit;
                s_tf[o >> 2] = (unsigned char)(t | STAGE_USED);
            }
        };
        // a wavefront's lists (every fourth): one sweep over the stage entries' bits counts
        // them, a second one writes those that fit
        constexpr int LPW = GROUPS / (BLOCK / WAVE);
        auto sweep = [&](auto write_tag, int g0, int g1, int (&nl)[LPW], int (&np)[LPW], const int (&pf)[LPW], const int (&pb)[LPW]) {
            constexpr bool WRITE = decltype(write_tag)::value;
            unsigned nbits = lane < kept ? s_om[lane] : 0u;
            int ntype = s_tf[lane];
            for (int k0 = 0; k0 < kept; k0 += WAVE) {
                const int k = k0 + lane;
                const unsigned bits = nbits;
                const bool lip = (ntype & 3) == 0;
                const int kn = min(k + WAVE, USTAGE - 1);                // the next entries are on their way
                nbits = k + WAVE < kept ? s_om[kn] : 0u;
                ntype = s_tf[kn];
#pragma unroll
                for (int j = 0; j < LPW; ++j) {
                    const int g = wv + j * (BLOCK / WAVE);
                    if (g < g0 || g >= g1) continue;                     // wavefront-uniform
                    const bool in = (bits >> g) & 1u;
                    const unsigned long long ml = __ballot(in && lip), mp = __ballot(in && !lip);
                    if constexpr (WRITE) {
                        const unsigned long long mine = lip ? ml : mp;
                        const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(mine >> 32),
                                                                     __builtin_amdgcn_mbcnt_lo((unsigned)mine, 0u));
                        const int at = lip ? pf[j] + nl[j] + before : pb[j] - 1 - np[j] - before;
                        if (in) s_list[at] = (uint16_t)(4 * k);
                    }
                    nl[j] += __popcll(ml);
                    np[j] += __popcll(mp);
                }
            }
        };
        {
            int nl[LPW] = {0, 0, 0, 0}, np[LPW] = {0, 0, 0, 0};
            sweep(std::false_type{}, 0, G, nl, np, nl, np);
#pragma unroll
            for (int j = 0; j < LPW; ++j) {
                const int g = wv + j * (BLOCK / WAVE);
                if (lane == 0 && g < G) {
                    s_nl[g] = (uint16_t)nl[j];
                    s_np[g] = (uint16_t)np[j];
                }
            }
        }
        for (int g0 = 0; g0 < G;) {
            __syncthreads();
            // the lists' places: whole groups of four entries, with room for both ends' padding
            if (wv == 0) {
                const bool has = lane < G - g0;
                const int x = wave_incl_scan(has ? (((int)s_nl[g0 + lane] + (int)s_np[g0 + lane] + 3) & ~3) + 4 : 0);
                if (lane < GROUPS) s_lofs[lane + 1] = x;
                const unsigned long long fit = __ballot(has && x <= CLIST);
                if (lane == 0) {
                    s_lofs[0] = 0;
                    s_nfit = __popcll(fit);                              // x grows with the lane: a prefix
                }
            }
            static_assert(CLIST >= USTAGE + 8, "one list always fits");
            __syncthreads();
            const int nfit = s_nfit;
            {
                int nl[LPW] = {0, 0, 0, 0}, np[LPW] = {0, 0, 0, 0}, pf[LPW], pb[LPW];
#pragma unroll
                for (int j = 0; j < LPW; ++j) {
                    const int g = min(max(wv + j * (BLOCK / WAVE) - g0, 0), nfit - 1);
                    pf[j] = __builtin_amdgcn_readfirstlane(s_lofs[g]);
                    pb[j] = __builtin_amdgcn_readfirstlane(s_lofs[g + 1]);
                }
                sweep(std::true_type{}, g0, g0 + nfit, nl, np, pf, pb);
#pragma unroll
                for (int j = 0; j < LPW; ++j) {
                    const int g = wv + j * (BLOCK / WAVE);
                    if (g >= g0 && g < g0 + nfit && lane < 3) {          // the last groups of four end in valid offsets
                        s_list[pf[j] + nl[j] + lane] = 0;
                        s_list[pb[j] - 1 - np[j] - lane] = 0;
                    }
                }
            }
            __syncthreads();
            if (valid && mygrp >= g0 && mygrp < g0 + nfit) {
                const int nl = s_nl[mygrp], np = s_np[mygrp], wl = (nl + 31) >> 5;
                const int pf = s_lofs[mygrp - g0], pb = s_lofs[mygrp - g0 + 1];    // lipids from pf up, proteins from pb - 1 down
                auto scan = [&](auto per_tag) {
                    constexpr bool PER = decltype(per_tag)::value;
                    auto dist2 = [&](int o) {
                        float dx = ux(o) - oix, dy = uy(o) - oiy, dz = uz(o) - oiz;
                        if constexpr (PER) {
                            dx -= Lx * rintf(dx * iLx);
                            dy -= Ly * rintf(dy * iLy);
                            dz -= Lz * rintf(dz * iLz);
                        }
                        return dx * dx + dy * dy + dz * dz;
                    };
                    // the hits among 32 candidates of a segment from candidate c on (n in all),
                    // candidate c + b in bit b, four candidates per trip
                    auto word = [&](auto lip_tag, int c, int n) {
                        constexpr bool LIP = decltype(lip_tag)::value;
                        const int ne = min(32, n - c);
                        unsigned m = 0u;
#pragma unroll 2
                        for (int j = 0; j < ne; j += 4) {
                            const uint2 l = *reinterpret_cast<const uint2 *>(s_list + (LIP ? pf + c + j : pb - 4 - c - j));
                            const int o[4] = {(int)(l.x & 0xffffu), (int)(l.x >> 16), (int)(l.y & 0xffffu), (int)(l.y >> 16)};
                            m >>= 4;
#pragma unroll
                            for (int q = 0; q < 4; ++q) {
                                const int oq = o[LIP ? q : 3 - q];
                                const float rl = LIP ? rlA : sel3f(s_tf[oq >> 2] & 3, rlA, rlB, rlC);
                                const bool hit = dist2(oq) < rl && oq != oself;
                                m |= hit ? 1u << (28 + q) : 0u;
                            }
                        }
                        m >>= 32 - ((ne + 3) & ~3);
                        return ne < 32 ? m & ((1u << ne) - 1u) : m;
                    };
                    // candidate b of word w in the list
                    auto at = [&](int w, int b) { return w < wl ? pf + 32 * w + b : pb - 1 - 32 * (w - wl) - b; };
                    // a row's test against the pruned radius
                    auto inner = [&](int o, int t) { return dist2(o) < sel3f(t, riA, riB, riC); };
                    // hit words, the empty ones left out; their numbers, five bits each, in wix
                    const int nw = wl + ((np + 31) >> 5);
                    int w = 0, slots = 0;
                    unsigned long long wix = 0ull;
                    for (; w < nw && w < 32 && slots < MWORDS; ++w) {
                        const unsigned m = w < wl ? word(std::true_type{}, 32 * w, nl) : word(std::false_type{}, 32 * (w - wl), np);
                        if (m) {
                            s_m[slots * BLOCK + tid] = m;
                            wix |= (unsigned long long)w << (5 * slots);
                            ++slots;
                            cnt += __popc(m);
                        }
                    }
                    // rows: every lane's next hit, eight rows to a store
                    const int n = min(cnt, MAXNB);
                    // (the next three words wait in registers; a group that uses up more reads on)
                    int slot = 0;
                    unsigned cur = n > 0 ? s_m[tid] : 0u;
                    for (int g = 0; __ballot(8 * g < n) != 0ull; ++g) {
                        int o[8], t[8];
                        bool have[8];
                        unsigned e[8], pbits = 0u;
                        unsigned n1 = s_m[min(slot + 1, MWORDS - 1) * BLOCK + tid], n2 = s_m[min(slot + 2, MWORDS - 1) * BLOCK + tid],
                                 n3 = s_m[min(slot + 3, MWORDS - 1) * BLOCK + tid];
                        const int last3 = slot + 3;
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            have[q] = 8 * g + q < n;
                            const bool next = have[q] && cur == 0u;
                            slot += next ? 1 : 0;
                            cur = next ? n1 : cur;
                            n1 = next ? n2 : n1;
                            n2 = next ? n3 : n2;
                            if (__builtin_expect(__ballot(next && slot > last3) != 0ull, 0))
                                if (next && slot > last3) cur = s_m[slot * BLOCK + tid];
                            const int cw = (int)(wix >> (5 * slot)) & 31;
                            o[q] = have[q] ? at(cw, __ffs(cur) - 1) : pf;
                            cur &= cur - 1u;
                        }
#pragma unroll
                        for (int q = 0; q < 8; ++q) o[q] = s_list[o[q]];
#pragma unroll
                        for (int q = 0; q < 8; ++q) t[q] = s_tf[o[q] >> 2] & 3;
                        bool in[8];
#pragma unroll
                        for (int q = 0; q < 8; ++q) in[q] = have[q] && inner(o[q], t[q]);
#pragma unroll
                        for (int q = 0; q < 8; ++q) {
                            e[q] = have[q] ? (unsigned)(o[q] >> 2) : 0xffffu;
                            if (in[q]) {
                                pbits |= 1u << q;
                                s_tf[o[q] >> 2] = (unsigned char)(t[q] | STAGE_USED);
                            }
                        }
                        const v4u out = {e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
                        stg(row8 + g * CHUNK, out);
                        const unsigned pw = pbits << (8 * (g & 3));
                        if (g < 4) pm0 |= pw;
                        else if (g < 8) pm1 |= pw;
                        else pm2 |= pw;
                        mygroups = g + 1;
                    }
                    // the words beyond the slots, hit by hit
                    for (; w < nw; ++w) {
                        unsigned m = w < wl ? word(std::true_type{}, 32 * w, nl) : word(std::false_type{}, 32 * (w - wl), np);
                        for (; m; m &= m - 1u, ++cnt) {
                            if (cnt >= MAXNB) continue;
                            const int o1 = s_list[at(w, __ffs(m) - 1)], t1 = s_tf[o1 >> 2] & 3;
                            if ((cnt & 7) == 0) {
                                stg(row8 + (cnt >> 3) * CHUNK, v4u{~0u, ~0u, ~0u, ~0u});
                                mygroups = (cnt >> 3) + 1;
                            }
                            stg(row + nl_at(cnt, lane), (uint16_t)(o1 >> 2));
                            if (inner(o1, t1)) {
                                const unsigned bit = 1u << (cnt & 31);
                                if (cnt < 32) pm0 |= bit;
                                else if (cnt < 64) pm1 |= bit;
                                else pm2 |= bit;
                                s_tf[o1 >> 2] = (unsigned char)(t1 | STAGE_USED);
                            }
                        }
                    }
                };
                if (periodic) scan(std::true_type{});
                else scan(std::false_type{});
                // more than a list holds: once more, hit by hit, at the next level's radius (the
                // code stays small: the kernel's loops run from the instruction cache)
                float ra = rlA, rb = rlB, rc = rlC;
#pragma unroll 1
                while (__builtin_expect(cnt > MAXNB && level < NL_LEVELS, 0)) {
                    ++level;
                    auto shorter = [&](float r2) {
                        const float r = sqrtf(r2) - P.nl_step;
                        return r * r;
                    };
                    ra = shorter(ra);
                    rb = shorter(rb);
                    rc = shorter(rc);
                    cnt = mygroups = 0;
                    pm0 = pm1 = pm2 = 0u;
#pragma unroll 1
                    for (int c = 0; c < nl + np; ++c) {
                        const int o = s_list[c < nl ? pf + c : pb - 1 - (c - nl)], t = s_tf[o >> 2] & 3;
                        const float d2 = dist2f(ux(o), uy(o), uz(o), oix, oiy, oiz);
                        if (!(d2 < sel3f(t, ra, rb, rc)) || o == oself) continue;
                        if (cnt < MAXNB) {
                            if ((cnt & 7) == 0) {
                                stg(row8 + (cnt >> 3) * CHUNK, v4u{~0u, ~0u, ~0u, ~0u});
                                mygroups = (cnt >> 3) + 1;
                            }
                            stg(row + nl_at(cnt, lane), (uint16_t)(o >> 2));
                            if (d2 < sel3f(t, riA, riB, riC)) {
                                const unsigned bit = 1u << (cnt & 31);
                                if (cnt < 32) pm0 |= bit;
                                else if (cnt < 64) pm1 |= bit;
                                else pm2 |= bit;
                                s_tf[o >> 2] = (unsigned char)(t | STAGE_USED);
                            }
                        }
                        ++cnt;
                    }
                }
            }
            g0 += nfit;
        }
    }
    int32_t *col = S.nl + (size_t)(chunk_ok ? chunk : 0) * MAXNB * CHUNK + lane;
    if (!staged && valid) {
        double cut0 = P.rl2[ti][0], cut1 = P.rl2[ti][1], cut2 = P.rl2[ti][2];
        for (;;) {
            cnt = 0;
            // the paired cells whose sphere reaches this particle, four side by side, and their
            // members likewise
            constexpr int SB = 4;
            const int qe = S.cnbr_start[A + 1];
            for (int q0 = S.cnbr_start[A]; q0 < qe; q0 += SB) {
                int b[SB], e[SB];
#pragma unroll
                for (int k = 0; k < SB; ++k) {
                    const int B = ldg(S.cnbr + min(q0 + k, qe - 1));
                    const D4 c = ldg(S.seed + B);
                    b[k] = ldg(S.cstart + B);
                    e[k] = b[k] + ldg(S.ccount + B);
                    double dx, dy, dz;
                    const double d2 = dist2_exact(S, pi.x, pi.y, pi.z, c.x, c.y, c.z, dx, dy, dz);
                    const double reach = c.w + P.cell_search + 1e-9;
                    if (q0 + k >= qe || d2 > reach * reach) e[k] = b[k];
                }
                for (int k = 0; k < SB; ++k)
                    for (int j0 = b[k]; j0 < e[k]; j0 += SB) {
                        D4 pj[SB];
#pragma unroll
                        for (int h = 0; h < SB; ++h) pj[h] = ldpos(S, min(j0 + h, e[k] - 1));
#pragma unroll
                        for (int h = 0; h < SB; ++h) {
                            const int j = j0 + h;
                            double dx, dy, dz;
                            const double d2 = dist2_exact(S, pi.x, pi.y, pi.z, pj[h].x, pj[h].y, pj[h].z, dx, dy, dz);
                            if (j < e[k] && j != i && d2 < (pj[h].w == 0.0 ? cut0 : (pj[h].w == 1.0 ? cut1 : cut2))) {
                                if (cnt < MAXNB) stg(col + cnt * CHUNK, (int32_t)j);
                                ++cnt;
                            }
                        }
                    }
            }
            if (cnt <= MAXNB || level == NL_LEVELS) break;
            ++level;
            auto shorter = [&](double r2) {
                const double r = sqrt(r2) - (double)P.nl_step;
                return r * r;
            };
            cut0 = shorter(cut0);
            cut1 = shorter(cut1);
            cut2 = shorter(cut2);
        }
    }
    int rows = wave_max_int(cnt);
    const int wlevel = wave_max_int(level);
    if (wlevel > 0 && lane == 0) {
        atomicOr(&S.sc->err, rows > MAXNB ? ERR_NLIST | ERR_NPAIRS : ERR_NLIST);
        atomicMax(&S.sc->level, wlevel);
    }
    rows = min(rows, MAXNB);
    if (chunk_ok && lane == 0) S.nlk[chunk] = rows;
    if (lane == 0) s_rows[wv] = rows;
    int nkept = -1;
    if (staged) {
        // pad every lane to the chunk's groups of rows, then the pruned stage and lists
        if (chunk_ok)
            for (int g = mygroups; 8 * g < rows; ++g) stg(row8 + g * CHUNK, v4u{~0u, ~0u, ~0u, ~0u});
        uint2 *s_bp = reinterpret_cast<uint2 *>(s_raw);
        nkept = pruned_stage(S, lb, kept, s_tf, s_bp, s_w);
        constexpr int PAIRS = (sizeof(s_raw) - 8 * (SMAX / 32)) / (4 * BLOCK);
        if (chunk_ok)
            emit_pruned<PAIRS>(S, chunk, rows, pm0, pm1, pm2, s_bp, reinterpret_cast<uint16_t *>(s_raw + 8 * (SMAX / 32)));
    } else if (chunk_ok) {
        // a block without a stage walks its 32-bit lists unpruned
        const int mycnt = valid ? min(cnt, MAXNB) : 0;
        for (int r = mycnt; r < rows; ++r) stg(col + r * CHUNK, (int32_t)-1);
        if (lane == 0) S.ilk[chunk] = rows;
    }
    __syncthreads();
    if (tid == 0) {
        S.scount[lb] = staged ? kept : -1;
        S.iscount[lb] = nkept;
        const int m = max(max(s_rows[0], s_rows[1]), max(s_rows[2], s_rows[3]));
        if (m > 0) max_if_larger(&S.sc->nlrows, m);             // the build's longest list
    }
}

void launch_nlist(const LaunchCtx &L) {
    hipLaunchKernelGGL(k_nlist, dim3(L.nblk_p), dim3(BLOCK), 0, L.st, L.S, L.maps, L.prm);
}

// ------------------------------------------------------------------ pruned lists

// One block per 256 consecutive cell-sorted particles.  The block's lists hold every
// partner within rc + 2 skin at the last build; the partners within rc + 2 inner skin
// are kept in a pruned list, which the force kernel walks instead.  The build writes
// the pruned lists for its own positions; this kernel prunes again between builds, at
// the current positions.  A pair left out was farther apart than rc + 2 inner
// skin when the lists were pruned, so it cannot come within rc before some particle
// has moved more than the inner skin since then; the runtime prunes again before
// that.  As in the list build, the test runs on FP32 offsets from the block's first
// particle against the radius widened by 1e-3 sigma (offsets are limited to 4096
// sigma), so the pruned list is a superset of the exact neighbour set; blocks whose
// offsets exceed that keep every entry.  The partners kept form the block's pruned
// stage (in stage order); the pruned list holds indices into it, padded with 0xffff.
// Blocks without a stage (32-bit global lists) are not pruned (pruned count -1).
// Every particle's current position becomes its reference for the displacement
// since the prune.
__global__ __launch_bounds__(BLOCK) void k_prune(const SysDev *Sd, Maps L_maps, DevParams P) {
    SYS_FROM(p);
    // the stage's offsets; after the test, the pruned stage's words and the row buffer
    __shared__ __align__(16) unsigned char s_raw[3 * SMAX * 4];
    __shared__ __align__(16) unsigned char s_tf[SMAX];     // type | STAGE_USED
    __shared__ int s_w[4];
    __shared__ int s_far[BLOCK / WAVE];
    float *s_x = reinterpret_cast<float *>(s_raw), *s_y = s_x + SMAX, *s_z = s_y + SMAX;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int chunk = lb * (BLOCK / WAVE) + wv;
    const bool chunk_ok = chunk < S.nchunk;
    const int i = lb * BLOCK + tid;
    const bool valid = i < S.n;
    const D4 pi = valid ? ldpos(S, i) : D4{0.0, 0.0, 0.0, 0.0};
    if (valid) S.xp[i] = F3{(float)pi.x, (float)pi.y, (float)pi.z};
    const int scnt = S.scount[lb];
    const int rows = chunk_ok ? __builtin_amdgcn_readfirstlane(min(S.nlk[chunk], MAXNB)) : 0;
    if (scnt < 0) {
        if (chunk_ok && lane == 0) S.ilk[chunk] = rows;
        if (tid == 0) S.iscount[lb] = -1;
        return;
    }
    const D4 ref = ld3(S.pos + (size_t)lb * BLOCK);
    bool far = false;
    // eight entries per thread in flight: their slots, then their positions
    for (int q0 = tid; q0 < scnt; q0 += 8 * BLOCK) {
        int slot[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int q = q0 + k * BLOCK;
            slot[k] = q < scnt ? ldg(S.stage + (size_t)lb * SSTRIDE + q) : -1;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int q = q0 + k * BLOCK;
            if (slot[k] < 0) break;
            const V3 pj = ldg(S.pos + stage_slot(slot[k]));
            const float ox = (float)minimg1(pj.x - ref.x, S.per[0], S.box[0]);
            const float oy = (float)minimg1(pj.y - ref.y, S.per[1], S.box[1]);
            const float oz = (float)minimg1(pj.z - ref.z, S.per[2], S.box[2]);
            s_x[q] = ox;
            s_y[q] = oy;
            s_z[q] = oz;
            s_tf[q] = (unsigned char)stage_type(slot[k]);
            far = far || !(fabsf(ox) <= LIST_EXTENT && fabsf(oy) <= LIST_EXTENT && fabsf(oz) <= LIST_EXTENT);
        }
    }
    // the bytes up to the next whole word of flags
    if (tid < 32 && scnt + tid < ((scnt + 31) & ~31)) s_tf[scnt + tid] = 0;
    const bool any_far = __ballot(far) != 0ull;      // offsets out of range or not finite
    if (lane == 0) s_far[wv] = any_far;
    __syncthreads();
    const bool keep_all = (s_far[0] | s_far[1] | s_far[2] | s_far[3]) != 0;
    const v4u *src = reinterpret_cast<const v4u *>(S.nl16 + (size_t)(chunk_ok ? chunk : 0) * MAXNB * CHUNK) + lane;
    unsigned pm0 = 0u, pm1 = 0u, pm2 = 0u;           // the rows that stay
    static_assert(MAXNB == 96, "row bits in three words");
    if (valid && chunk_ok) {
        const int ti = (int)pi.w;
        const float oix = (float)minimg1(pi.x - ref.x, S.per[0], S.box[0]);
        const float oiy = (float)minimg1(pi.y - ref.y, S.per[1], S.box[1]);
        const float oiz = (float)minimg1(pi.z - ref.z, S.per[2], S.box[2]);
        const float rA = ti == 0 ? P.rin2f[0][0] : (ti == 1 ? P.rin2f[1][0] : P.rin2f[2][0]);
        const float rB = ti == 0 ? P.rin2f[0][1] : (ti == 1 ? P.rin2f[1][1] : P.rin2f[2][1]);
        const float rC = ti == 0 ? P.rin2f[0][2] : (ti == 1 ? P.rin2f[1][2] : P.rin2f[2][2]);
        const bool periodic = (S.per[0] | S.per[1] | S.per[2]) != 0;
        const float Lx = S.per[0] ? (float)S.box[0] : 0.0f, Ly = S.per[1] ? (float)S.box[1] : 0.0f,
                    Lz = S.per[2] ? (float)S.box[2] : 0.0f;
        const float iLx = S.per[0] ? 1.0f / Lx : 0.0f, iLy = S.per[1] ? 1.0f / Ly : 0.0f,
                    iLz = S.per[2] ? 1.0f / Lz : 0.0f;
        const int ng = (rows + 7) / 8;
        v4u nx0 = {~0u, ~0u, ~0u, ~0u}, nx1 = nx0;   // the next two groups of eight rows
        if (ng > 0) nx0 = ldg(src);
        if (ng > 1) nx1 = ldg(src + CHUNK);
        for (int g = 0; g < ng; ++g) {
            const v4u e = nx0;
            nx0 = nx1;
            if (g + 2 < ng) nx1 = ldg(src + (g + 2) * CHUNK);
            unsigned pbits = 0u;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const int k = (int)((q & 1) ? e[q >> 1] >> 16 : e[q >> 1] & 0xffffu);
                const bool real = k < scnt;          // 0xffff pads
                const int ks = real ? k : 0;
                float dx = s_x[ks] - oix, dy = s_y[ks] - oiy, dz = s_z[ks] - oiz;
                if (periodic) {
                    dx -= Lx * rintf(dx * iLx);
                    dy -= Ly * rintf(dy * iLy);
                    dz -= Lz * rintf(dz * iLz);
                }
                const float d2 = dx * dx + dy * dy + dz * dz;
                const int t = s_tf[ks] & 3;
                if (real && (keep_all || d2 < sel3f(t, rA, rB, rC))) {
                    pbits |= 1u << q;
                    s_tf[ks] = (unsigned char)(t | STAGE_USED);
                }
            }
            const unsigned pw = pbits << (8 * (g & 3));
            if (g < 4) pm0 |= pw;
            else if (g < 8) pm1 |= pw;
            else pm2 |= pw;
        }
    }
    uint2 *s_bp = reinterpret_cast<uint2 *>(s_raw);
    const int nkept = pruned_stage(S, lb, scnt, s_tf, s_bp, s_w);
    constexpr int PAIRS = (sizeof(s_raw) - 8 * (SMAX / 32)) / (4 * BLOCK);
    if (chunk_ok)
        emit_pruned<PAIRS>(S, chunk, rows, pm0, pm1, pm2, s_bp, reinterpret_cast<uint16_t *>(s_raw + 8 * (SMAX / 32)));
    if (tid == 0) S.iscount[lb] = nkept;
}

// Block map of the systems in the mask (particle blocks only), for prunes outside a
// cell update.  One block of MAX_SLOTS threads.
__global__ __launch_bounds__(MAX_SLOTS) void k_mask_maps(const SysDev *Sd, int nsys, unsigned long long m0,
                                                         unsigned long long m1, unsigned long long m2,
                                                         unsigned long long m3, int32_t *out) {
    __shared__ int s_w[16];
    const int s = threadIdx.x;
    int cnt = 0;
    if (s < nsys) {
        const unsigned long long w = (s < 64) ? m0 : (s < 128) ? m1 : (s < 192) ? m2 : m3;
        if ((w >> (s & 63)) & 1ull) cnt = (Sd[s].n + BLOCK - 1) / BLOCK;
    }
    int tot;
    const int ex = block_excl_scan(cnt, s_w, tot);
    if (s <= nsys) out[s] = ex;
}

void launch_prune(const LaunchCtx &L) {
    if (L.nblk_p > 0) hipLaunchKernelGGL(k_prune, dim3(L.nblk_p), dim3(BLOCK), 0, L.st, L.S, L.maps, L.prm);
}

void launch_mask_maps(const LaunchCtx &L, const unsigned long long m[4], int32_t *out) {
    hipLaunchKernelGGL(k_mask_maps, dim3(1), dim3(MAX_SLOTS), 0, L.st, L.S, L.nsys, m[0], m[1], m[2], m[3], out);
}

// ------------------------------------------------------------------ entry points used by the runtime

void launch_set_rebuild(const LaunchCtx &L, const unsigned long long m[4], int32_t *out) {
    hipLaunchKernelGGL(k_set_rebuild, dim3(1), dim3(MAX_SLOTS), 0, L.st, L.S, L.nsys, m[0], m[1], m[2], m[3], out);
}

// Seeds from the lipids, and their grid.
void launch_init_seeds(const LaunchCtx &L, const int32_t *const *lipids) {
    hipLaunchKernelGGL(k_init_seeds, dim3(L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps, lipids);
    hipLaunchKernelGGL(k_seed_bbox_partial, dim3(L.nblk_c), dim3(BLOCK), 0, L.st, L.S, L.maps);
    grid_build(L, 1);
}

void launch_pack(const LaunchCtx &L, int s, const double *x, const double *n, const int32_t *type,
                 const double *v, const double *w, int count) {
    hipLaunchKernelGGL(k_pack_multi, dim3((count + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, L.st, L.S, s, x, n, type,
                       v, w);
}

}  // namespace rbc

// Many-sphere rigid-body run with pairwise capillary-bridge forces from the learned surrogate.
// See include/pf_dem.h for the model; the kernels of a step are
//   k_dem_cells       one block: the spheres sorted by cell (runs large enough for a cell grid);
//   k_dem_search      one wave per sphere: bridged partners in ascending index order, their count and
//                     the count of partners with a larger index, from the cells or from all spheres;
//   k_dem_rows        four lanes per sphere: exclusive scan of the upper counts (one network row per
//                     bridge i < j, ordered by (i, j)), bridge features and network inputs;
//   the network       on the rows counted on the device (no host round trip inside a step);
//   k_dem_forces      sixteen lanes per sphere: bridge and contact forces summed in partner order,
//                     and the semi-implicit Euler step with periodic wrap into the other state buffer.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <string>
#include <vector>

#include "../../include/pf_dem.h"

// the network's stream, input width and batch limit (mlp.hip)
__attribute__((visibility("hidden"))) void pfm_internal_info(const pf_mlp *h, int *n_in, int *max_batch,
                                                             void **stream);
// forward pass of *n_dev rows (at most max_rows), the count read on the device; false when the network's
// width has no such pass (mlp.hip)
__attribute__((visibility("hidden"))) bool pfm_internal_forward_counted(pf_mlp *h, const float *x, int max_rows,
                                                                        const int *n_dev, float *y);

namespace pfd {

constexpr int MAX_OVERRIDES = 256;
constexpr double PI = 3.14159265358979323846;

struct DemDev {
    int n, cap, max_pairs, n_over;
    double L, dt, density, kn, gn, theta, cfrac, gmin, gmax;
    float ish[4], isc[4], osh, osc;
    const double *R;
    double *x, *v, *F;    // state the step reads
    double *xn, *vn;      // state it writes
    int *nbr, *deg, *nup, *off;
    int nc;               // cells per edge of the search grid, 0: every pair is tested
    int *cell;            // cell of each sphere
    int *cstart, *cidx;   // first slot of each cell (nc^3 + 1), sphere of each slot
    // two bridge lists of max_pairs rows: the rows of an evaluation go to the one that ctl[3] does not name
    int *pij;
    double *pfeat, *pforce;
    float *X;
    const float *Y;
    // [0] bridges of the current evaluation, [1] error bits (1: neighbours, 2: pairs; once set, the
    // steps that follow change nothing), [2] bridges of the last evaluation without an error and [3] its
    // list (0 or 1)
    int *ctl;
    const int *over_ij;
    const double *over_f;
};

// minimum image; x_j - x_i and x_i - x_j give exactly negated results, and the surface gap is
// formed as r - (R_i + R_j), so "bridged" is symmetric in (i, j) to the bit
__device__ __forceinline__ double mimg(double d, double L) { return d - L * floor(d / L + 0.5); }

// Cells per edge at most: 4096 counters in LDS.
constexpr int MAX_NC = 16;
// spheres from which the cell grid is used
constexpr int CELL_MIN_N = 2048;

// cell coordinate of x, in [0, L) unless the sphere moved so far (more than 2^53 boxes) in the step that
// the wrap rounded: then that of its image in the box, which its minimum images belong to
__device__ __forceinline__ int cell_of(double x, double scale, int nc) {
    double t = x * scale;
    if (!(t >= 0.0 && t < nc)) t -= nc * floor(t / nc);
    return min(nc - 1, max(0, (int)t));
}

// index of the cell of a sphere at x, y, z
__device__ __forceinline__ int cell_index(double x, double y, double z, double scale, int nc) {
    return cell_of(x, scale, nc) + nc * (cell_of(y, scale, nc) + nc * cell_of(z, scale, nc));
}

// cell of every sphere (the start state; the Euler step keeps them current)
__global__ __launch_bounds__(256) void k_dem_assign(DemDev p) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < p.n) p.cell[i] = cell_index(p.x[3 * i], p.x[3 * i + 1], p.x[3 * i + 2], p.nc / p.L, p.nc);
}

// Spheres sorted by cell: counts in LDS, scan, slots by LDS counters (the order inside a cell does not
// matter: the search sorts its few partners by index), the sorted list assembled in LDS and written
// in order.  One block of 1024 threads; thread t owns spheres t, t + 1024, ..  One block because a wider
// sort is several launches; it touches 4 bytes of a sphere each way (writing the positions in cell order
// here, one line per lane and store, took 48 us at 12000 spheres).
__global__ __launch_bounds__(1024) void k_dem_cells(DemDev p) {
    constexpr int PER = 16;  // n <= 16384
    __shared__ int cnt[MAX_NC * MAX_NC * MAX_NC], part[16];
    __shared__ unsigned short order[1024 * PER];
    const int t = threadIdx.x, nc = p.nc, n3 = nc * nc * nc;
    int cell[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) cell[k] = t + 1024 * k < p.n ? p.cell[t + 1024 * k] : -1;
    for (int c = t; c < n3; c += 1024) cnt[c] = 0;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (cell[k] >= 0) atomicAdd(&cnt[cell[k]], 1);
    __syncthreads();
    // exclusive scan: four counters a thread, waves, waves' totals
    int v[4], s = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[j] = 4 * t + j < n3 ? cnt[4 * t + j] : 0;
        s += v[j];
    }
    int inc = s;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int u = __shfl_up(inc, off, 64);
        if ((t & 63) >= off) inc += u;
    }
    if ((t & 63) == 63) part[t >> 6] = inc;
    __syncthreads();
    int o = inc - s;
    for (int w = 0; w < (t >> 6); ++w) o += part[w];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (4 * t + j < n3) {
            cnt[4 * t + j] = o;
            p.cstart[4 * t + j] = o;
            o += v[j];
        }
    if (t == 0) p.cstart[n3] = p.n;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (cell[k] >= 0) order[atomicAdd(&cnt[cell[k]], 1)] = (unsigned short)(t + 1024 * k);
    __syncthreads();
    for (int i = t; i < p.n; i += 1024) p.cidx[i] = order[i];
}

// Is j a bridged partner of i?  A cheap test (reciprocal, no root) with a margin far above its rounding
// passes the few candidates on to the definition.
__device__ __forceinline__ bool bridged(const DemDev &p, double invL, double xi, double yi, double zi, double Ri,
                                        double xj, double yj, double zj, double Rj) {
    const double ax = xj - xi, ay = yj - yi, az = zj - zi;
    const double bx = ax - p.L * floor(ax * invL + 0.5), by = ay - p.L * floor(ay * invL + 0.5),
                 bz = az - p.L * floor(az * invL + 0.5);
    const double reach = (Ri + Rj + p.gmax) * (1.0 + 1e-9) + 1e-12 * p.L;
    if (bx * bx + by * by + bz * bz > reach * reach) return false;
    const double dx = mimg(ax, p.L), dy = mimg(ay, p.L), dz = mimg(az, p.L);
    return sqrt(dx * dx + dy * dy + dz * dz) - (Ri + Rj) < p.gmax;
}

// Partners of every sphere, one wave each.  CELLS: the 27 cells around the sphere's (a cell is at least
// as wide as the longest bridge, so no partner lies outside), two lanes per cell; the partners, at
// most 64, are put in index order by counting.  Else every sphere, 256 a round, in index order.
// The cells pay from a few thousand spheres (below, the sort's own launch costs more than it saves).
template <bool CELLS>
__global__ __launch_bounds__(256) void k_dem_search(DemDev p) {
    __shared__ int found[4][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int w = blockIdx.x * 4 + wave;
    if (w >= p.n) return;  // whole wave
    const double invL = 1.0 / p.L;
    int i, cnt = 0, up = 0;
    const unsigned long long below = (1ull << lane) - 1ull;
    if constexpr (CELLS) {
        i = p.cidx[w];
        const double xi = p.x[3 * i], yi = p.x[3 * i + 1], zi = p.x[3 * i + 2], Ri = p.R[i];
        const int nc = p.nc, k = lane >> 1;  // neighbour cell
        int s = 0, e = 0;
        if (k < 27) {
            auto wrap = [&](int c) { return c < 0 ? c + nc : (c >= nc ? c - nc : c); };
            const int c0 = p.cell[i], c = wrap(c0 % nc + k % 3 - 1) +
                                          nc * (wrap((c0 / nc) % nc + (k / 3) % 3 - 1) + nc * wrap(c0 / (nc * nc) + k / 9 - 1));
            s = p.cstart[c] + (lane & 1);
            e = p.cstart[c + 1];
        }
        while (__ballot(s < e)) {
            bool b = false;
            int j = i;
            if (s < e) {
                j = p.cidx[s];
                b = j != i && bridged(p, invL, xi, yi, zi, Ri, p.x[3 * j], p.x[3 * j + 1], p.x[3 * j + 2], p.R[j]);
            }
            const unsigned long long m = __ballot(b);
            const int rank = cnt + __popcll(m & below);
            if (b && rank < 64) found[wave][rank] = j;
            cnt += __popcll(m);
            up += __popcll(__ballot(b && j > i));
            s += 2;
        }
        __builtin_amdgcn_wave_barrier();
        const int have = min(cnt, 64);
        if (lane < have) {
            const int j = found[wave][lane];
            int rank = 0;
            for (int m = 0; m < have; ++m) rank += found[wave][m] < j ? 1 : 0;
            if (rank < p.cap) p.nbr[(long long)i * p.cap + rank] = j;
        }
    } else {
        i = w;
        const double xi = p.x[3 * i], yi = p.x[3 * i + 1], zi = p.x[3 * i + 2], Ri = p.R[i];
        for (int base = 0; base < p.n; base += 256) {
            double xj[4], yj[4], zj[4], Rj[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = min(base + 64 * u + lane, p.n - 1);
                xj[u] = p.x[3 * j];
                yj[u] = p.x[3 * j + 1];
                zj[u] = p.x[3 * j + 2];
                Rj[u] = p.R[j];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int j = base + 64 * u + lane;
                const bool b = j < p.n && j != i && bridged(p, invL, xi, yi, zi, Ri, xj[u], yj[u], zj[u], Rj[u]);
                const unsigned long long m = __ballot(b);
                const int rank = cnt + __popcll(m & below);
                if (b && rank < p.cap) p.nbr[(long long)i * p.cap + rank] = j;
                cnt += __popcll(m);
                up += __popcll(__ballot(b && j > i));
            }
        }
    }
    if (lane == 0) {
        p.deg[i] = min(cnt, p.cap);
        p.nup[i] = up;
        if (cnt > p.cap) atomicOr(p.ctl + 1, 1);
    }
}

__device__ __forceinline__ void bridge_features(const DemDev &p, double Ri, double Rj, double gap, double *f,
                                                double *rstar) {
    const double rs = 2.0 * Ri * Rj / (Ri + Rj);
    const double vl = p.cfrac / (1.0 - p.cfrac) * (4.0 / 3.0) * PI * (Ri * Ri * Ri + Rj * Rj * Rj);
    f[0] = fmax(gap, p.gmin) / rs;
    f[1] = fmin(Ri, Rj) / fmax(Ri, Rj);
    f[2] = vl / (rs * rs * rs);
    f[3] = p.theta;
    *rstar = rs;
}

// Network rows of the bridges (i, j > i), 64 spheres a block and four lanes each.  A block sums the
// upper counts of all spheres before its own (at most 64 KB, from L2) instead of waiting for a scan of
// its own launch.
__global__ __launch_bounds__(256) void k_dem_rows(DemDev p) {
    __shared__ int part[4], offs[64];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int i0 = blockIdx.x * 64;
    int s = 0;
    for (int k = 4 * tid; k < i0; k += 1024) {
        const int4 v = *(const int4 *)(p.nup + k);  // i0 is a multiple of 64
        s += (v.x + v.y) + (v.z + v.w);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (lane == 0) part[wave] = s;
    __syncthreads();
    const int first = (part[0] + part[1]) + (part[2] + part[3]);
    if (wave == 0) {
        const int u = i0 + lane < p.n ? p.nup[i0 + lane] : 0;
        int inc = u;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const int t = __shfl_up(inc, off, 64);
            if (lane >= off) inc += t;
        }
        offs[lane] = first + inc - u;
        if (i0 + lane < p.n) p.off[i0 + lane] = first + inc - u;
        if (blockIdx.x == gridDim.x - 1 && lane == 63) {
            p.ctl[0] = first + inc;
            if (first + inc > p.max_pairs) atomicOr(p.ctl + 1, 2);
        }
    }
    __syncthreads();
    const int i = i0 + (tid >> 2);
    if (i >= p.n) return;
    const double xi = p.x[3 * i], yi = p.x[3 * i + 1], zi = p.x[3 * i + 2], Ri = p.R[i];
    const int deg = p.deg[i], lower = deg - p.nup[i], list = p.ctl[3] ^ 1;
    for (int k = max(lower, 0) + (tid & 3); k < deg; k += 4) {
        const int j = p.nbr[(long long)i * p.cap + k];
        const int row = offs[tid >> 2] + (k - lower);
        if (j < i || row >= p.max_pairs) continue;
        const double dx = mimg(p.x[3 * j] - xi, p.L), dy = mimg(p.x[3 * j + 1] - yi, p.L),
                     dz = mimg(p.x[3 * j + 2] - zi, p.L);
        const double gap = sqrt(dx * dx + dy * dy + dz * dz) - (Ri + p.R[j]);
        double f[4], rs;
        bridge_features(p, Ri, p.R[j], gap, f, &rs);
        const int out = row + list * p.max_pairs;
        p.pij[2 * out] = i;
        p.pij[2 * out + 1] = j;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            p.pfeat[4 * (long long)out + c] = f[c];
            p.X[4 * (long long)row + c] = (float)((f[c] - (double)p.ish[c]) * (double)p.isc[c]);
        }
    }
}

// Forces, sixteen lanes per sphere (one partner each, then the next sixteen), summed in partner order;
// with move != 0 the Euler step into the other state buffer.  The evaluation's bridge list becomes the
// current one.  After an error the state is carried over unchanged and nothing else is written.
__global__ __launch_bounds__(256) void k_dem_forces(DemDev p, int move) {
    const int i = blockIdx.x * 16 + (threadIdx.x >> 4), q = threadIdx.x & 15;
    const bool err = p.ctl[1] != 0;
    if (blockIdx.x == 0 && threadIdx.x == 0 && !err) {
        p.ctl[2] = p.ctl[0];
        p.ctl[3] ^= 1;
    }
    const bool in = i < p.n;
    const int is = in ? i : 0;
    const double xi = p.x[3 * is], yi = p.x[3 * is + 1], zi = p.x[3 * is + 2], Ri = p.R[is];
    const double vxi = p.v[3 * is], vyi = p.v[3 * is + 1], vzi = p.v[3 * is + 2];
    const int di = in && !err ? p.deg[is] : 0, lower_i = di - p.nup[is];
    double Fx = 0.0, Fy = 0.0, Fz = 0.0;
    for (int k0 = 0; __ballot(k0 < di); k0 += 16) {
        const int k = k0 + q;
        double fn = 0.0, ex = 0.0, ey = 0.0, ez = 0.0;
        bool on = k < di;
        if (on) {
            const int j = p.nbr[(long long)i * p.cap + k];
            const double dx = mimg(p.x[3 * j] - xi, p.L), dy = mimg(p.x[3 * j + 1] - yi, p.L),
                         dz = mimg(p.x[3 * j + 2] - zi, p.L);
            const double r = sqrt(dx * dx + dy * dy + dz * dz);
            const double Rj = p.R[j], gap = r - (Ri + Rj);
            ex = dx / r;
            ey = dy / r;
            ez = dz / r;
            // network row of the bridge (min(i, j), max(i, j)); a lower partner's list is searched eight
            // entries a round
            int row = p.off[i] + (k - lower_i);
            if (j < i) {
                const int dj = p.deg[j];
                int pos = dj;
                for (int s = 0; s < dj && pos == dj; s += 8) {
                    int v[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) v[u] = p.nbr[(long long)j * p.cap + min(s + u, dj - 1)];
#pragma unroll
                    for (int u = 7; u >= 0; --u)
                        if (s + u < dj && v[u] == i) pos = s + u;
                }
                on = pos < dj;  // always: the gap is symmetric in (i, j) to the bit
                row = p.off[j] + (pos - (dj - p.nup[j]));
            }
            if (on) {
                const double rs = 2.0 * Ri * Rj / (Ri + Rj);
                double Fb = ((double)p.Y[row] * (double)p.osc + (double)p.osh) * rs;
                const int a = min(i, j), b = max(i, j);
                for (int o = 0; o < p.n_over; ++o)
                    if (p.over_ij[2 * o] == a && p.over_ij[2 * o + 1] == b) Fb = p.over_f[o];
                if (j > i) p.pforce[row] = Fb;
                fn = Fb;  // along e (towards j)
                if (gap < 0.0) {
                    const double vn = (p.v[3 * j] - vxi) * ex + (p.v[3 * j + 1] - vyi) * ey + (p.v[3 * j + 2] - vzi) * ez;
                    fn += p.kn * gap + p.gn * vn;
                }
            }
        }
        for (int s = 0; s < 16 && __ballot(k0 + s < di); ++s) {
            const double f = __shfl(fn, s, 16), gx = __shfl(ex, s, 16), gy = __shfl(ey, s, 16), gz = __shfl(ez, s, 16);
            if (__shfl((int)on, s, 16)) {
                Fx += f * gx;
                Fy += f * gy;
                Fz += f * gz;
            }
        }
    }
    if (!in || q >= 3) return;
    const double F = q == 0 ? Fx : (q == 1 ? Fy : Fz), xq = q == 0 ? xi : (q == 1 ? yi : zi),
                 vq = q == 0 ? vxi : (q == 1 ? vyi : vzi);
    if (!err) p.F[3 * i + q] = F;
    if (!move) return;
    double v = vq, x = xq;
    if (!err) {
        const double inv_m = 1.0 / (p.density * (4.0 / 3.0) * PI * Ri * Ri * Ri);
        v = vq + F * inv_m * p.dt;
        x = xq + v * p.dt;
        x -= p.L * floor(x / p.L);
        if (x >= p.L) x -= p.L;  // x / L rounded up to 1
    }
    p.vn[3 * i + q] = v;
    p.xn[3 * i + q] = x;
    if (p.nc) {
        // the cell of the new position, from the three lanes that hold its coordinates
        const double x0 = __shfl(x, 0, 16), x1 = __shfl(x, 1, 16), x2 = __shfl(x, 2, 16);
        if (q == 0) p.cell[i] = cell_index(x0, x1, x2, p.nc / p.L, p.nc);
    }
}

}  // namespace pfd

using namespace pfd;

struct pf_dem {
    pf_dem_config cfg;
    hipStream_t stream = nullptr;
    pf_mlp *net = nullptr;
    char *ws = nullptr;
    DemDev d{};
    int *ctl_host = nullptr;  // pinned, 4 ints
    int last_pairs = 0, last_list = 0;  // bridges of the last evaluation without an error, and its list
    std::string err;
};

namespace {

thread_local std::string g_dem_init_error;

int dfail(pf_dem *h, int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    if (h)
        h->err = buf;
    else
        g_dem_init_error = buf;
    return code;
}

#define DCHK(h, call)                                                                              \
    do {                                                                                           \
        hipError_t e_ = (call);                                                                    \
        if (e_ != hipSuccess) return dfail((h), PF_LBM_EDEVICE, "%s: %s", #call, hipGetErrorString(e_)); \
    } while (0)

int blocks(int n, int per) { return (n + per - 1) / per; }

}  // namespace

extern "C" {

int pf_dem_init(const pf_dem_config *cfg, const double *radii, const double *x0, const double *v0, pf_mlp *net,
                void *workspace, size_t ws_bytes, void *hip_stream, pf_dem **out, size_t *ws_bytes_needed) {
    g_dem_init_error.clear();
    if (!cfg) return dfail(nullptr, PF_LBM_EINVAL, "cfg is NULL");
    if (cfg->struct_size < sizeof(pf_dem_config)) return dfail(nullptr, PF_LBM_EINVAL, "bad struct_size");
    if (cfg->n < 2 || cfg->n > 16384) return dfail(nullptr, PF_LBM_EINVAL, "n must be in [2, 16384]");
    if (cfg->max_neighbours < 1 || cfg->max_neighbours > 64)
        return dfail(nullptr, PF_LBM_EINVAL, "max_neighbours must be in [1, 64]");
    if (cfg->max_pairs < 1 || cfg->max_pairs > 65536) return dfail(nullptr, PF_LBM_EINVAL, "max_pairs in [1, 65536]");
    if (!(cfg->dt > 0) || !(cfg->density > 0) || !(cfg->k_n >= 0) || !(cfg->gamma_n >= 0))
        return dfail(nullptr, PF_LBM_EINVAL, "dt and density must be positive, k_n and gamma_n non-negative");
    if (!(cfg->theta >= 0 && cfg->theta <= 0.5 * PI)) return dfail(nullptr, PF_LBM_EINVAL, "theta must be in [0, pi/2]");
    if (!(cfg->liquid_fraction > 0 && cfg->liquid_fraction < 1))
        return dfail(nullptr, PF_LBM_EINVAL, "liquid_fraction must be in (0, 1)");
    if (!(cfg->gap_min >= 0 && cfg->gap_max > cfg->gap_min)) return dfail(nullptr, PF_LBM_EINVAL, "need 0 <= gap_min < gap_max");
    const int n = cfg->n, cap = cfg->max_neighbours, P = cfg->max_pairs;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = (off + bytes + 255) / 256 * 256;
        return o;
    };
    const size_t oR = take(8 * (size_t)n), ox = take(24 * (size_t)n), ov = take(24 * (size_t)n),
                 ox2 = take(24 * (size_t)n), ov2 = take(24 * (size_t)n), ocst = take(4 * (size_t)(MAX_NC * MAX_NC * MAX_NC + 1)),
                 ocidx = take(4 * (size_t)n), ocell = take(4 * (size_t)n),
                 oF = take(24 * (size_t)n), onbr = take(4 * (size_t)n * cap), odeg = take(4 * (size_t)n),
                 onup = take(4 * (size_t)n), ooff = take(4 * (size_t)n), opij = take(16 * (size_t)P),
                 opfeat = take(64 * (size_t)P), opforce = take(8 * (size_t)P), oX = take(16 * (size_t)P),
                 oY = take(4 * (size_t)P), octl = take(16), oover = take(8 * MAX_OVERRIDES),
                 overf = take(8 * MAX_OVERRIDES);
    if (ws_bytes_needed) *ws_bytes_needed = off;
    if (!workspace) return PF_LBM_OK;
    if (!out || !radii || !x0 || !v0 || !net) return dfail(nullptr, PF_LBM_EINVAL, "NULL argument");
    if (ws_bytes < off) return dfail(nullptr, PF_LBM_ENOMEM, "workspace of %zu bytes, %zu needed", ws_bytes, off);
    if ((uintptr_t)workspace % 256) return dfail(nullptr, PF_LBM_EINVAL, "workspace must be 256-byte aligned");
    int n_in = 0, max_batch = 0;
    void *net_stream = nullptr;
    pfm_internal_info(net, &n_in, &max_batch, &net_stream);
    if (n_in != 4) return dfail(nullptr, PF_LBM_EINVAL, "the network must take 4 inputs (it takes %d)", n_in);
    if (max_batch < P) return dfail(nullptr, PF_LBM_EINVAL, "network max_batch %d below max_pairs %d", max_batch, P);
    if (net_stream != hip_stream) return dfail(nullptr, PF_LBM_EINVAL, "the network is bound to another stream");
    double rmax = 0.0;
    for (int i = 0; i < n; ++i) {
        if (!(radii[i] > 0)) return dfail(nullptr, PF_LBM_EINVAL, "radius %d is not positive", i);
        rmax = std::max(rmax, radii[i]);
        for (int c = 0; c < 3; ++c)
            if (!(x0[3 * i + c] >= 0 && x0[3 * i + c] < cfg->box) || !std::isfinite(v0[3 * i + c]))
                return dfail(nullptr, PF_LBM_EINVAL, "sphere %d: position outside [0, box) or velocity not finite", i);
    }
    if (!(cfg->box > 4.0 * rmax + 2.0 * cfg->gap_max))
        return dfail(nullptr, PF_LBM_EINVAL, "box must exceed 4 max radius + 2 gap_max (unique minimum image)");
    pf_dem *h = new (std::nothrow) pf_dem;
    if (!h) return dfail(nullptr, PF_LBM_ENOMEM, "host allocation failed");
    h->cfg = *cfg;
    h->stream = (hipStream_t)hip_stream;
    h->net = net;
    h->ws = (char *)workspace;
    DemDev &d = h->d;
    d.n = n;
    d.cap = cap;
    d.max_pairs = P;
    d.n_over = 0;
    d.L = cfg->box;
    d.dt = cfg->dt;
    d.density = cfg->density;
    d.kn = cfg->k_n;
    d.gn = cfg->gamma_n;
    d.theta = cfg->theta;
    d.cfrac = cfg->liquid_fraction;
    d.gmin = cfg->gap_min;
    d.gmax = cfg->gap_max;
    for (int c = 0; c < 4; ++c) {
        d.ish[c] = cfg->in_shift[c];
        d.isc[c] = cfg->in_scale[c];
    }
    d.osh = cfg->out_shift;
    d.osc = cfg->out_scale;
    char *w = h->ws;
    d.R = (const double *)(w + oR);
    d.x = (double *)(w + ox);
    d.v = (double *)(w + ov);
    d.F = (double *)(w + oF);
    d.xn = (double *)(w + ox2);
    d.vn = (double *)(w + ov2);
    d.cstart = (int *)(w + ocst);
    d.cidx = (int *)(w + ocidx);
    d.cell = (int *)(w + ocell);
    // cells as wide as the longest possible bridge (a part in 10^9 wider, above the rounding of the
    // coordinates), at least three per edge so that the 27 around a sphere are distinct
    const double reach = (2.0 * rmax + cfg->gap_max) * (1.0 + 1e-9);
    const int nc = (int)std::min((double)MAX_NC, std::floor(cfg->box / reach));
    d.nc = nc >= 3 && n >= CELL_MIN_N ? nc : 0;
    d.nbr = (int *)(w + onbr);
    d.deg = (int *)(w + odeg);
    d.nup = (int *)(w + onup);
    d.off = (int *)(w + ooff);
    d.pij = (int *)(w + opij);
    d.pfeat = (double *)(w + opfeat);
    d.pforce = (double *)(w + opforce);
    d.X = (float *)(w + oX);
    d.Y = (const float *)(w + oY);
    d.ctl = (int *)(w + octl);
    d.over_ij = (const int *)(w + oover);
    d.over_f = (const double *)(w + overf);
    auto fail_init = [&](int rc) {
        g_dem_init_error = h->err;
        if (h->ctl_host) (void)hipHostFree(h->ctl_host);
        delete h;
        return rc;
    };
    if (hipHostMalloc((void **)&h->ctl_host, 16, hipHostMallocDefault) != hipSuccess) {
        h->ctl_host = nullptr;
        return fail_init(dfail(h, PF_LBM_EDEVICE, "hipHostMalloc failed"));
    }
    if (hipMemsetAsync(h->ws, 0, off, h->stream) != hipSuccess ||
        hipMemcpyAsync((void *)d.R, radii, 8 * (size_t)n, hipMemcpyHostToDevice, h->stream) != hipSuccess ||
        hipMemcpyAsync(d.x, x0, 24 * (size_t)n, hipMemcpyHostToDevice, h->stream) != hipSuccess ||
        hipMemcpyAsync(d.v, v0, 24 * (size_t)n, hipMemcpyHostToDevice, h->stream) != hipSuccess)
        return fail_init(dfail(h, PF_LBM_EDEVICE, "upload failed"));
    if (d.nc) k_dem_assign<<<blocks(n, 256), 256, 0, h->stream>>>(d);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(h->stream) != hipSuccess)
        return fail_init(dfail(h, PF_LBM_EDEVICE, "upload failed"));
    *out = h;
    return PF_LBM_OK;
}

}  // extern "C"

namespace {

// the kernels of one evaluation, with move the Euler step; nothing is waited for unless the network's
// width has no device-counted pass
int enqueue_evaluation(pf_dem *h, bool move) {
    DemDev &d = h->d;
    if (d.nc) {
        k_dem_cells<<<1, 1024, 0, h->stream>>>(d);
        k_dem_search<true><<<blocks(d.n, 4), 256, 0, h->stream>>>(d);
    } else {
        k_dem_search<false><<<blocks(d.n, 4), 256, 0, h->stream>>>(d);
    }
    k_dem_rows<<<blocks(d.n, 64), 256, 0, h->stream>>>(d);
    DCHK(h, hipGetLastError());
    if (!pfm_internal_forward_counted(h->net, d.X, d.max_pairs, d.ctl, (float *)d.Y)) {
        DCHK(h, hipMemcpyAsync(h->ctl_host, d.ctl, 16, hipMemcpyDeviceToHost, h->stream));
        DCHK(h, hipStreamSynchronize(h->stream));
        const int P = std::min(h->ctl_host[0], d.max_pairs);
        if (P > 0 && !h->ctl_host[1]) {
            const int rc = pf_mlp_forward(h->net, d.X, P, (float *)d.Y);
            if (rc != PF_LBM_OK) return dfail(h, rc, "network: %s", pf_mlp_last_error(h->net));
        }
    }
    k_dem_forces<<<blocks(d.n, 16), 256, 0, h->stream>>>(d, move ? 1 : 0);
    DCHK(h, hipGetLastError());
    if (move) {
        std::swap(d.x, d.xn);
        std::swap(d.v, d.vn);
    }
    return PF_LBM_OK;
}

// n evaluations with motion, or one without (n < 0); one wait, at the end
int run_evaluations(pf_dem *h, int n) {
    // refused before anything is enqueued where the wait at the end would be: the steps exchange the
    // state's two buffers as they are enqueued, and captured ones do not run
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    DCHK(h, hipStreamIsCapturing(h->stream, &cap));
    if (cap != hipStreamCaptureStatusNone)
        return dfail(h, PF_LBM_EDEVICE, "the run waits for its stream, which is being captured");
    DCHK(h, hipMemsetAsync(h->d.ctl + 1, 0, 4, h->stream));
    int rc = PF_LBM_OK;
    for (int s = 0; s < std::max(n, 1) && rc == PF_LBM_OK; ++s) rc = enqueue_evaluation(h, n > 0);
    // also where a step could not be enqueued: those before it have exchanged the lists
    DCHK(h, hipMemcpyAsync(h->ctl_host, h->d.ctl, 16, hipMemcpyDeviceToHost, h->stream));
    DCHK(h, hipStreamSynchronize(h->stream));
    h->last_pairs = h->ctl_host[2];
    h->last_list = h->ctl_host[3];
    if (rc != PF_LBM_OK) return rc;
    if (h->ctl_host[1] & 1) return dfail(h, PF_LBM_ENOMEM, "a sphere has more than max_neighbours bridged partners");
    if (h->ctl_host[1] & 2)
        return dfail(h, PF_LBM_ENOMEM, "%d bridges exceed max_pairs %d", h->ctl_host[0], h->d.max_pairs);
    return PF_LBM_OK;
}

}  // namespace

extern "C" {

int pf_dem_evaluate(pf_dem *h) {
    if (!h) return dfail(nullptr, PF_LBM_EINVAL, "handle is NULL");
    return run_evaluations(h, -1);
}

int pf_dem_step(pf_dem *h, int32_t n_steps) {
    if (!h) return dfail(nullptr, PF_LBM_EINVAL, "handle is NULL");
    if (n_steps < 0) return dfail(h, PF_LBM_EINVAL, "n_steps must be >= 0");
    return n_steps > 0 ? run_evaluations(h, n_steps) : PF_LBM_OK;
}

int pf_dem_state(pf_dem *h, double *x, double *v, double *f) {
    if (!h) return dfail(nullptr, PF_LBM_EINVAL, "handle is NULL");
    const size_t b = 24 * (size_t)h->d.n;
    if (x) DCHK(h, hipMemcpyAsync(x, h->d.x, b, hipMemcpyDeviceToHost, h->stream));
    if (v) DCHK(h, hipMemcpyAsync(v, h->d.v, b, hipMemcpyDeviceToHost, h->stream));
    if (f) DCHK(h, hipMemcpyAsync(f, h->d.F, b, hipMemcpyDeviceToHost, h->stream));
    DCHK(h, hipStreamSynchronize(h->stream));
    return PF_LBM_OK;
}

int pf_dem_pairs(pf_dem *h, int32_t max_out, int32_t *ij, double *features, double *force, int32_t *n_out) {
    if (!h || !n_out) return dfail(h, PF_LBM_EINVAL, "NULL argument");
    if (max_out < 0) return dfail(h, PF_LBM_EINVAL, "max_out must be >= 0");
    const int k = std::min(max_out, h->last_pairs);
    *n_out = h->last_pairs;
    if (k > 0) {
        const size_t row0 = (size_t)h->last_list * h->d.max_pairs;
        if (ij) DCHK(h, hipMemcpyAsync(ij, h->d.pij + 2 * row0, 8 * (size_t)k, hipMemcpyDeviceToHost, h->stream));
        if (features)
            DCHK(h, hipMemcpyAsync(features, h->d.pfeat + 4 * row0, 32 * (size_t)k, hipMemcpyDeviceToHost, h->stream));
        if (force) DCHK(h, hipMemcpyAsync(force, h->d.pforce, 8 * (size_t)k, hipMemcpyDeviceToHost, h->stream));
    }
    DCHK(h, hipStreamSynchronize(h->stream));
    return PF_LBM_OK;
}

int pf_dem_set_overrides(pf_dem *h, int32_t n, const int32_t *ij, const double *force) {
    if (!h) return dfail(nullptr, PF_LBM_EINVAL, "handle is NULL");
    if (n < 0 || n > MAX_OVERRIDES) return dfail(h, PF_LBM_EINVAL, "n must be in [0, %d]", MAX_OVERRIDES);
    if (n > 0 && (!ij || !force)) return dfail(h, PF_LBM_EINVAL, "NULL argument");
    std::vector<int> pairs(2 * (size_t)n);
    for (int k = 0; k < n; ++k) {
        const int a = ij[2 * k], b = ij[2 * k + 1];
        if (a < 0 || b < 0 || a >= h->d.n || b >= h->d.n || a == b || !std::isfinite(force[k]))
            return dfail(h, PF_LBM_EINVAL, "override %d: bad pair or force", k);
        pairs[2 * k] = std::min(a, b);
        pairs[2 * k + 1] = std::max(a, b);
    }
    if (n > 0) {
        DCHK(h, hipMemcpyAsync((void *)h->d.over_ij, pairs.data(), 8 * (size_t)n, hipMemcpyHostToDevice, h->stream));
        DCHK(h, hipMemcpyAsync((void *)h->d.over_f, force, 8 * (size_t)n, hipMemcpyHostToDevice, h->stream));
    }
    DCHK(h, hipStreamSynchronize(h->stream));
    h->d.n_over = n;
    return PF_LBM_OK;
}

void pf_dem_destroy(pf_dem *h) {
    if (!h) return;
    if (h->ctl_host) (void)hipHostFree(h->ctl_host);
    delete h;
}

const char *pf_dem_last_error(const pf_dem *h) { return h ? h->err.c_str() : g_dem_init_error.c_str(); }

}  // extern "C"

// FP64 ray shooting with the far field of the star sum as local (Taylor)
// expansions; a faster route to the sum of Eq. (3) for many stars.
//
// In complex notation (z = theta_x + i theta_y) the star term of Eq. (3) is
// alpha_x - i alpha_y = f(z) = sum_k m_k / (z - z_k).  Around a centre c,
// for a star with |c - z_k| > |z - c|,
//   m_k / (z - z_k) = sum_{q>=0} m_k u_k (-u_k rho)^q s^q,  u_k = 1/(c - z_k),
// with s = (z - c) / rho, so the far stars of a region add up to one
// polynomial F(s) = sum_q B_q s^q (the scaling by the region's radius rho
// keeps every |B_q| below sum m_k |u_k| theta_open^q, whatever the lattice
// spacing).  A star is far when |c - z_k| > rho / theta_open, with rho the
// region's radius (centre to corner ray): then every ray of the region has
// |(z - c) / (c - z_k)| <= theta_open and truncating after kOrder terms
// leaves an error below theta_open^(kOrder+1) (1 + theta_open) /
// (1 - theta_open) times m_k / |z - z_k| per star (1.5e-15 for
// theta_open = 0.25).  Near stars are summed directly, in index order.  The
// paper cites hierarchical tree codes as the way to avoid the brute-force
// sum (Sec. 1); this is a two-level form of that idea, on the ray side,
// whose truncation error stays at the level of FP64 rounding.
//
// Two levels.  The lattice is cut into blocks of L x L ray tiles (a tile is
// 4096 rays, 64 x 64 or a rectangle).  One workgroup per block expands the
// stars far from the whole block once (every star is visited once per block,
// not once per tile), keeping the block's near stars in lists.  Then a second
// kernel re-centres the block's polynomial on each tile (the shift of a
// polynomial is exact algebra: no new truncation), re-tests only the block's
// near stars (those far from the tile join its polynomial, the rest are
// summed directly), re-centres the tile's polynomial on 16 patches of 256
// rays, and evaluates those (Horner), adds the near stars and bins the rays.
// With L = 1 the block is the tile and the second test is skipped.  If a
// block has more near stars than its lists hold, its tiles sum every star
// directly.
//
// The block pass is a kernel of its own (expansion_block_kernel), which
// leaves each block's polynomial and near lists in a workspace for the
// tile kernel (expansion_tile_kernel); each runs at the occupancy its own
// registers allow.
//
// Star cells.  Optionally the stars are sorted once by the cell of a
// regular grid, and each cell gets a multipole expansion of its stars
// (M_j = sum_k m_k ((z_k - z_c) / r_c)^j).  The block pass then takes every
// cell far enough from the block, (r_c + rho) / theta_open or more between
// centres, through one multipole-to-local translation, and tests only the
// stars of the other cells one by one: the cell expansion of distant stars
// that tree codes rest on, at the same truncation bound per cell.
#include <algorithm>
#include <cmath>
#include <vector>

#include "ray_common.h"

namespace raysh {

namespace {

constexpr int kOrder = 24;            // Taylor terms B_0 .. B_kOrder
constexpr int kWaves = kThreads / 64;
constexpr int kNearPerWave = 512;     // near-star list capacity of each wave
constexpr int kBlockNear = kWaves * kNearPerWave;   // near stars of a block whose lists hold
// A tile is 4096 rays, 64 x 64 for a lattice of square cells, for others
// 64 / 2^k by 64 * 2^k (expansion_tiles).  A patch is a quarter of the tile
// either way.
constexpr int kPatchRays = 256;       // 16 x 16 / 2^k by 16 * 2^k
constexpr int kPatchSide = 4;         // patches along a tile's sides
constexpr int kPatches = kPatchSide * kPatchSide;
static_assert(kPatches * kPatchRays == kTileRays, "a tile's patches");
constexpr int kPatchOrder = 14;       // Taylor terms of a patch's polynomial (see expansion_tile_kernel)
constexpr int kTileNear = 256;        // near stars a tile keeps as a list of its own
constexpr int kCellMaxRows = kThreads;   // star-cell grid rows and columns: one thread per row
constexpr int kCellMaxCells = 4096;
constexpr int64_t kCellMaxStars = int64_t(1) << 26;   // the host keeps two copies while building
constexpr int32_t kCellMaxPerCell = 1 << 20;          // stars of one cell (its multipoles take one thread)

struct ExpShared {
    double2 A[kOrder + 1];                      // the block's coefficients
    double2 part[kWaves][kOrder + 1];           // per-wave partial sums
    int outer_idx[kWaves][kNearPerWave];        // the block's near stars, each wave's in index order
    int outer_n[kWaves];
    int row_lo[kCellMaxRows], row_hi[kCellMaxRows];   // each star-cell row's band of open cells
    int row_first[kCellMaxRows];                      // first record of the band's stars
    int row_pref[kCellMaxRows];                       // the bands' stars before this row
    int wave_tot[kWaves];
};

// What a block's pass over the stars leaves for its tiles: the block's
// coefficients and its near stars, each wave's list in order (the counts
// include stars beyond the lists' capacity).
struct BlockFar {
    double2 A[kOrder + 1];
    int outer_n[kWaves];
    int outer_idx[kWaves][kNearPerWave];
};

__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(__builtin_fma(a.x, b.x, -a.y * b.y), __builtin_fma(a.x, b.y, a.y * b.x));
}

// Centre and radius (centre to corner ray, slightly enlarged) of the rectangle
// of w x h lattice points whose first point is (i, j) of the block.
__device__ __forceinline__ void region(const ShootParams &p, int64_t i, int64_t j, int w, int h, double &cx,
                                       double &cy, double &rho) {
    const double x_first = image_angle(p.x0, p.i0 + i, p.dx);
    const double x_last = image_angle(p.x0, p.i0 + i + w - 1, p.dx);
    const double y_first = image_angle(p.y0, p.j0 + j, p.dy);
    const double y_last = image_angle(p.y0, p.j0 + j + h - 1, p.dy);
    cx = 0.5 * (x_first + x_last);
    cy = 0.5 * (y_first + y_last);
    const double hx = 0.5 * (x_last - x_first), hy = 0.5 * (y_last - y_first);
    rho = __builtin_sqrt(hx * hx + hy * hy) * (1.0 + 1e-12) + 1e-290;
}

// region() for a rectangle every lane of the wave shares: the results are
// moved to scalar registers.
__device__ __forceinline__ void region_uniform(const ShootParams &p, int64_t i, int64_t j, int w, int h, double &cx,
                                               double &cy, double &rho) {
    region(p, i, j, w, h, cx, cy, rho);
    cx = uniform_f64(cx);
    cy = uniform_f64(cy);
    rho = uniform_f64(rho);
}

// Maximum of a non-negative float over the wave, uniform.
__device__ __forceinline__ float wave_max(float v) {
#define RAYSH_DPP_MAX(ctrl, rows) \
    v = fmaxf(v, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), ctrl, rows, 0xf, true)))
    RAYSH_DPP_MAX(0x111, 0xf);   // row_shr 1, 2, 4, 8: lane 15 of each row of 16
    RAYSH_DPP_MAX(0x112, 0xf);
    RAYSH_DPP_MAX(0x114, 0xf);
    RAYSH_DPP_MAX(0x118, 0xf);
    RAYSH_DPP_MAX(0x142, 0xa);   // row_bcast 15 into rows 1 and 3
    RAYSH_DPP_MAX(0x143, 0xc);   // row_bcast 31 into rows 2 and 3
#undef RAYSH_DPP_MAX
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// The order at which a series in theta may stop: the smallest P with
// theta^(P + 1) <= 2^-56, at most `most` (theta2 = theta^2, uniform).
__device__ __forceinline__ int order_for(float theta2, int most) {
    const float l = -__log2f(theta2);   // +inf for 0
    const float P = 112.0f / l;
    return uniform(P >= 0.0f && P < (float)most ? (int)P : most);   // theta >= 1 or NaN: all terms
}

// One pass over `count` entries split into four contiguous quarters, one per
// wave.  fetch(e, k, x, y, m) gives entry e's star: its index k and record.
// A star farther than sqrt(r_near2) from (cx, cy) adds m u (-u rho)^q to
// the lane's coefficients; a nearer one is appended to its wave's out list,
// so that the concatenated out lists keep the entries' order.  out_n counts
// every near star, also beyond the capacity.
// SORTED: the stars come by cell.  Their fetches are longer (one is under way
// while the star before it is summed), and 64 of them lie close together, so
// the series stops at the order that the nearest one needs.  (Without an order
// the nearest of 64 needs most terms, and the tests and the registers, 222
// for 132, cost more: 16384 stars, 8192^2 rays 113 -> 138 us.)
template <bool SORTED, class Fetch>
__device__ __forceinline__ void p2l_pass(int count, Fetch fetch, double cx, double cy, double rho, double r_near2,
                                         double2 (&acc)[kOrder + 1], int (*out_idx)[kNearPerWave], int *out_n) {
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int per_wave = (count + kWaves - 1) / kWaves;
    const int w0 = uniform(wave * per_wave < count ? wave * per_wave : count);
    const int w1 = uniform(w0 + per_wave < count ? w0 + per_wave : count);
    int found = 0;   // this wave's near stars so far (uniform in the wave)
    int nk = 0;
    double nx = 0.0, ny = 0.0, nm = 0.0;
    if (SORTED && w0 + lane < w1) fetch(w0 + lane, nk, nx, ny, nm);
    for (int base = w0; base < w1; base += 64) {
        const bool valid = base + lane < w1;
        if (!SORTED && valid) fetch(base + lane, nk, nx, ny, nm);
        const int k = nk;
        const double sm = nm;
        const double dx = cx - nx, dy = cy - ny;
        const double d2 = dx * dx + dy * dy;
        if (SORTED && base + 64 + lane < w1) fetch(base + 64 + lane, nk, nx, ny, nm);
        const bool near = valid && d2 <= r_near2;
        const double inv = 1.0 / d2;
        int order = kOrder;
        if (SORTED) order = order_for(wave_max(valid && !near ? (float)(rho * rho * inv) : 0.0f), kOrder);
        if (valid && !near) {
            const double2 u = make_double2(dx * inv, -dy * inv);        // 1 / (c - z_k)
            const double2 mu = make_double2(-u.x * rho, -u.y * rho);    // -u rho
            double2 t = make_double2(sm * u.x, sm * u.y);               // m u
#pragma unroll
            for (int q = 0; q <= kOrder; ++q) {
                if (SORTED && q % 4 == 1 && q > order) break;
                acc[q].x += t.x;
                acc[q].y += t.y;
                if (q < kOrder) t = cmul(t, mu);
            }
        }
        const unsigned long long ball = __ballot(near);
        if (near) {
            const int pos = found + __popcll(ball & ((1ull << lane) - 1ull));
            if (pos < kNearPerWave) out_idx[wave][pos] = k;
        }
        found += __popcll(ball);
    }
    if (lane == 0) out_n[wave] = found;
}

// Binomial coefficients C(j + q, q) for j, q <= kOrder: exact integers (at
// most C(48, 24) < 2^53) built by Pascal's rule at compile time.
struct CellBinomialTable {
    double c[kOrder + 1][kOrder + 1];
};

constexpr CellBinomialTable make_cell_binomials() {
    CellBinomialTable t{};
    for (int j = 0; j <= kOrder; ++j)
        for (int q = 0; q <= kOrder; ++q)
            t.c[j][q] = (j == 0 || q == 0) ? 1.0 : t.c[j - 1][q] + t.c[j][q - 1];
    return t;
}

__constant__ CellBinomialTable kCellBinomial = make_cell_binomials();

// A star cell's multipole expansion (scaled: M_j = sum_k m_k ((z_k - z_c) / r_c)^j)
// translated to the local expansion of a region of centre C and radius
// rho, added to acc.  With D = C - z_c, w = 1/D and g = -rho w,
//   sum_k m_k / (C + rho s - z_k) = w sum_j M_j (r_c w)^j sum_q C(j + q, q) g^q s^q,
// which converges for (r_c + rho) < |D|.  The terms of total degree n = j + q
// add up to at most theta^n of the cell's field, theta = (r_c + rho) / |D|,
// those of one j to (a / (1 - g))^j and those of one q to (g / (1 - a))^q, with
// a = r_c / |D| and g = rho / |D| here; the sums stop where each bound is
// below 2^-56 for the wave's nearest cells (and at kOrder in j and in q), so
// what is dropped stays below theta^(kOrder+1) / (1 - theta), the bound of the
// per-star expansion.  A cell 14 r_c away takes 14 terms where all 25 x 25
// took 625.
__device__ __forceinline__ void m2l_cell(const double2 *M, double dx, double dy, double rc, double rho, bool active,
                                         double2 (&acc)[kOrder + 1]) {
    const double inv = 1.0 / (dx * dx + dy * dy);
    const float fa = wave_max(active ? (float)__builtin_sqrt(rc * rc * inv) : 0.0f);
    const float fg = wave_max(active ? (float)__builtin_sqrt(rho * rho * inv) : 0.0f);
    const auto sq = [](float x) { return x * x; };
    const int degree = order_for(sq(fa + fg), 2 * kOrder);
    const int most_j = min(order_for(sq(fa / (1.0f - fg)), kOrder), degree);
    const int most_q = order_for(sq(fg / (1.0f - fa)), kOrder);
    if (!active) return;
    const double2 w = make_double2(dx * inv, -dy * inv);
    const double2 g = make_double2(-rho * w.x, -rho * w.y);
    const double2 a = make_double2(rc * w.x, rc * w.y);
    double2 ap = w;   // w (r_c w)^j
    double2 m = M[0], m1 = M[min(1, most_j)];
    for (int j = 0; j <= most_j; ++j) {   // uniform trip count
        double2 t = cmul(m, ap);
        m = m1;
        m1 = M[min(j + 2, most_j)];   // two terms ahead: a lane's loads miss its L1
        const int last = min(most_q, degree - j);   // uniform
#pragma unroll
        for (int q = 0; q <= kOrder; ++q) {
            if (q % 2 == 1 && q > last) break;
            const double b = kCellBinomial.c[j][q];
            acc[q].x = __builtin_fma(b, t.x, acc[q].x);
            acc[q].y = __builtin_fma(b, t.y, acc[q].y);
            if (q < kOrder) t = cmul(t, g);
        }
        ap = cmul(ap, a);
    }
}

// Exclusive prefix sum of one int per thread over the workgroup (values of
// threads past `n` count as zero); returns the thread's prefix and writes the
// total to *total.  Every thread of the workgroup must call it.
__device__ __forceinline__ int block_exclusive_scan(int v, int *wave_tot, int *total) {
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    int incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int up = __shfl_up(incl, off, 64);
        if (lane >= off) incl += up;
    }
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < kWaves; ++w) {
        if (w < wave) before += wave_tot[w];
        all += wave_tot[w];
    }
    *total = all;
    return before + incl - v;
}

// The sum a lane keeps when lanes with bit W set take `upper` and the others
// `lower`, its own plus the one of its partner across that bit.
template <int W>
__device__ __forceinline__ double swap_halves(double lower, double upper) {
    const uint64_t a = __builtin_bit_cast(uint64_t, lower), b = __builtin_bit_cast(uint64_t, upper);
    typedef unsigned uint2v __attribute__((ext_vector_type(2)));
    uint2v lo, hi;
    if constexpr (W == 32) {
        lo = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
        hi = __builtin_amdgcn_permlane32_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
    } else {
        lo = __builtin_amdgcn_permlane16_swap((unsigned)a, (unsigned)b, false, false);
        hi = __builtin_amdgcn_permlane16_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
    }
    return __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]) +
           __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}

// Wave sum of the lanes' coefficients in a fixed order: lane l < 2 (kOrder + 1)
// returns real component l.  The components, padded with zeros to 64 slots,
// are reduced by recursive halving: at the step of lane mask m, lanes with
// that bit keep the upper half of their slots and the others the lower half,
// each adds the half its partner sends, so after six steps lane l holds the
// wave's sum of slot l (63 exchanges per lane instead of 300 for a butterfly
// over every slot).
__device__ __forceinline__ double wave_reduce_coeffs(const double2 (&acc)[kOrder + 1]) {
    constexpr int kSlots = 2 * (kOrder + 1);
    static_assert(kSlots <= 64, "one slot per lane at the end");
    const int lane = threadIdx.x % 64;
    double v[64];
#pragma unroll
    for (int q = 0; q <= kOrder; ++q) {
        v[2 * q] = acc[q].x;
        v[2 * q + 1] = acc[q].y;
    }
#pragma unroll
    for (int i = kSlots; i < 64; ++i) v[i] = 0.0;
    // lane bits 5 and 4: v_permlane*_swap exchanges the halves (rows) of two
    // registers, after which both hold what one lane is to add
#pragma unroll
    for (int i = 0; i < 32; ++i) v[i] = swap_halves<32>(v[i], v[i + 32]);
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] = swap_halves<16>(v[i], v[i + 16]);
#pragma unroll
    for (int n = 16; n > 1; n /= 2) {
        const int m = n / 2;                 // the lane bit of this step
        const bool upper = (lane & m) != 0;
#pragma unroll
        for (int i = 0; i < n / 2; ++i) {
            const double keep = upper ? v[i + n / 2] : v[i];
            const double send = upper ? v[i] : v[i + n / 2];
            v[i] = keep + __shfl_xor(send, m, 64);
        }
    }
    return v[0];
}

// Workgroup sum of the lanes' coefficients into dst: the waves' sums, added
// in turn.
__device__ __forceinline__ void reduce_coeffs(double2 (&acc)[kOrder + 1], ExpShared &ex, double2 *dst) {
    constexpr int kSlots = 2 * (kOrder + 1);
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const double v = wave_reduce_coeffs(acc);
    if (lane < kSlots) reinterpret_cast<double *>(&ex.part[wave][0])[lane] = v;
    __syncthreads();
    if (threadIdx.x < kSlots) {
        double t = reinterpret_cast<const double *>(&ex.part[0][0])[threadIdx.x];
        for (int w = 1; w < kWaves; ++w) t += reinterpret_cast<const double *>(&ex.part[w][0])[threadIdx.x];
        reinterpret_cast<double *>(dst)[threadIdx.x] = t;
    }
    __syncthreads();
}

// The block pass over star cells.  A cell whose centre is at least
// (r_c + rho) / theta_open from the block's centre enters the block's
// coefficients through its multipole expansion (m2l_cell); the rest form,
// in each row of the cell grid, a band of open cells whose stars are tested
// one by one as in the pass over every star, so the near lists hold the
// same stars (in cell order, index order within a cell).
__device__ __forceinline__ void block_pass_cells(const StarCells &cells, double bcx, double bcy, double brho,
                                                 double inv_theta, double r_near2, double2 (&acc)[kOrder + 1],
                                                 ExpShared &ex) {
    const int ncx = uniform(cells.ncx), ncy = uniform(cells.ncy);
    const double h = uniform_f64(cells.h), rc = uniform_f64(cells.rc);
    const double gx0 = uniform_f64(cells.gx0), gy0 = uniform_f64(cells.gy0);
    const double rmac = (rc + brho) * inv_theta;
    const double rmac2 = rmac * rmac;
    // row j (one thread each): its band [lo, hi] and the band's stars
    const int j = threadIdx.x;
    int first = 0, cnt = 0;
    if (j < ncy) {
        const double dy = bcy - (gy0 + ((double)j + 0.5) * h);
        int lo = ncx, hi = -1;
        for (int i = 0; i < ncx; ++i) {
            const double dx = bcx - (gx0 + ((double)i + 0.5) * h);
            if (dx * dx + dy * dy < rmac2) {
                if (lo > i) lo = i;
                hi = i;
            }
        }
        ex.row_lo[j] = lo;
        ex.row_hi[j] = hi;
        if (hi >= lo) {
            first = cells.start[j * ncx + lo];
            cnt = cells.start[j * ncx + hi + 1] - first;
        }
        ex.row_first[j] = first;
    }
    int total = 0;
    const int pref = block_exclusive_scan(cnt, ex.wave_tot, &total);   // its barrier publishes the bands
    if (j < ncy) ex.row_pref[j] = pref;
    __syncthreads();
    // every non-empty cell outside the bands, through its multipole expansion
    const int n_cells = ncx * ncy;
    for (int base = 0; base < n_cells; base += kThreads) {   // uniform
        const int c = base + threadIdx.x;
        bool far = false;
        int i = 0, jj = 0;
        if (c < n_cells) {
            i = c % ncx;
            jj = c / ncx;
            far = (i < ex.row_lo[jj] || i > ex.row_hi[jj]) && cells.start[c + 1] != cells.start[c];
        }
        const double dx = bcx - (gx0 + ((double)i + 0.5) * h);
        const double dy = bcy - (gy0 + ((double)jj + 0.5) * h);
        m2l_cell(cells.mult + (size_t)(far ? c : 0) * (kOrder + 1), dx, dy, rc, brho, far, acc);
    }
    // the bands' stars, one by one: entry e is in the last row whose prefix
    // is at most e (rows before it hold fewer stars, empty rows share their
    // successor's prefix); a lane's entries ascend, and so do their rows
    const Star *sorted = cells.sorted;
    int row = -1, row_end = 0, shift = 0;   // the row of the lane's last entry, the first entry past it
    p2l_pass<true>(
        uniform(total),
        [&](int e, int &k, double &x, double &y, double &m) {
            if (e >= row_end) {
                int lo = row < 0 ? 0 : row, hi = ncy - 1;
                while (lo < hi) {
                    const int mid = (lo + hi + 1) / 2;
                    if (ex.row_pref[mid] <= e) lo = mid;
                    else hi = mid - 1;
                }
                row = lo;
                row_end = lo + 1 < ncy ? ex.row_pref[lo + 1] : 0x7fffffff;
                shift = ex.row_first[lo] - ex.row_pref[lo];
            }
            const Star st = sorted[shift + e];
            x = st.x;
            y = st.y;
            m = st.m;
            k = (int)__builtin_bit_cast(long long, st.pad);
        },
        bcx, bcy, brho, r_near2, acc, ex.outer_idx, ex.outer_n);
}

// The block pass, one workgroup per block of block_w x block_h rays:
// the stars far from the block enter its local expansion A (through star
// cells when CELLS), the near ones go to its lists; both are written to
// far[blockIdx.x] for the tile kernel.  Two workgroups per compute unit: the
// cells' translations need the registers.  262144 stars, 2048^2 rays, one
// workgroup a unit: 104 -> 55 us with the series cut at the order that each
// wave's nearest cell or star needs, and the next star and multipoles fetched
// ahead (the multipoles' part: 117 -> 110 us a map); bound by VALU issue with
// one wave a SIMD, and latency.
template <bool CELLS>
__global__ __launch_bounds__(kThreads, 2) void expansion_block_kernel(ShootParams p, StarCells cells,
                                                                      double theta_open, int blocks_x,
                                                                      int block_w, int block_h,
                                                                      BlockFar *__restrict__ far) {
    __shared__ ExpShared ex;
    const int64_t b_i = (int64_t)(blockIdx.x % blocks_x) * block_w;
    const int64_t b_j = (int64_t)(blockIdx.x / blocks_x) * block_h;
    const ConstStar *st = const_stars(uniform_ptr(p.stars));
    const int n = uniform(p.n_stars);
    const double inv_theta = uniform_f64(1.0 / theta_open);
    double bcx, bcy, brho;
    region_uniform(p, b_i, b_j, block_w, block_h, bcx, bcy, brho);
    double2 acc[kOrder + 1];
#pragma unroll
    for (int q = 0; q <= kOrder; ++q) acc[q] = make_double2(0.0, 0.0);
    const double r_near = brho * inv_theta;
    const double r_near2 = uniform_f64(r_near * r_near);
    if constexpr (CELLS) {
        block_pass_cells(cells, bcx, bcy, brho, inv_theta, r_near2, acc, ex);
    } else {
        p2l_pass<false>(
            n,
            [&](int e, int &k, double &x, double &y, double &m) {
                k = e;
                x = st[e].x;
                y = st[e].y;
                m = st[e].m;
            },
            bcx, bcy, brho, r_near2, acc, ex.outer_idx, ex.outer_n);
    }
    reduce_coeffs(acc, ex, ex.A);   // its barriers also publish outer_n
    BlockFar *f = far + blockIdx.x;
    if (threadIdx.x <= kOrder) f->A[threadIdx.x] = ex.A[threadIdx.x];
    if (threadIdx.x < kWaves) f->outer_n[threadIdx.x] = ex.outer_n[threadIdx.x];
    for (int w = 0; w < kWaves; ++w) {
        const int cnt = min(ex.outer_n[w], kNearPerWave);
        for (int i = threadIdx.x; i < cnt; i += kThreads) f->outer_idx[w][i] = ex.outer_idx[w][i];
    }
}

// q!, q <= kOrder (rounded from 23! on).
struct FactorialTable {
    double f[kOrder + 1];
};

constexpr FactorialTable make_factorials() {
    FactorialTable t{};
    t.f[0] = 1.0;
    for (int q = 1; q <= kOrder; ++q) t.f[q] = t.f[q - 1] * q;
    return t;
}

__constant__ FactorialTable kFactorial = make_factorials();

// Re-centring.  A polynomial sum_q A_q s^q on s = a + b s' has the coefficients
//   B_r = b^r sum_{q >= r} A_q C(q, r) a^(q - r)
//       = (b^r / r!) sum_{j >= 0} alpha_{r + j} a^j / j!,  alpha_q = q! A_q,
// and the last sum by Horner takes one complex multiply-add a step:
//   S <- alpha_{r + j - 1} + (a / j) S,  j = kOrder - r ... 1.
// (Scaling by factorials takes the binomials out of the loop; re-centring is
// exact algebra, so no truncation enters beyond the coefficients dropped.)
// alpha is zero past kOrder, so a step from any larger j is harmless.
__device__ __forceinline__ double2 recentre_step(double2 S, double2 alpha, double ax, double ay) {
    return make_double2(__builtin_fma(S.x, ax, __builtin_fma(-S.y, ay, alpha.x)),
                        __builtin_fma(S.x, ay, __builtin_fma(S.y, ax, alpha.y)));
}

// 1 / q!.
constexpr FactorialTable make_inverse_factorials() {
    FactorialTable t = make_factorials();
    for (int q = 0; q <= kOrder; ++q) t.f[q] = 1.0 / t.f[q];
    return t;
}

__constant__ FactorialTable kInverseFactorial = make_inverse_factorials();

// 1 / j (f[0] unused).
constexpr FactorialTable make_inverses() {
    FactorialTable t{};
    t.f[0] = 0.0;
    for (int q = 1; q <= kOrder; ++q) t.f[q] = 1.0 / q;
    return t;
}

__constant__ FactorialTable kInverse = make_inverses();

// Steps j = hi ... lo of the coefficients r0, r0 + 4, ... (the first N of
// them; alpha points at alpha_r0).
template <int N, int EACH>
__device__ __forceinline__ void recentre_run(double2 (&S)[EACH], const double2 *alpha, double sx, double sy, int hi,
                                             int lo) {
#pragma unroll 2
    for (int j = hi; j >= lo; --j) {
        const double ax = sx * kInverse.f[j], ay = sy * kInverse.f[j];
#pragma unroll
        for (int i = 0; i < (N < EACH ? N : EACH); ++i) S[i] = recentre_step(S[i], alpha[kWaves * i + j - 1], ax, ay);
    }
}

__device__ __forceinline__ double int_pow(double b, int r) {
    double t = 1.0;
#pragma unroll
    for (int bit = 0; bit < 5; ++bit) {   // r <= kOrder < 32
        if (r & (1 << bit)) t *= b;
        b *= b;
    }
    return t;
}

constexpr int kComputeUnits = 256;
constexpr int kTilesPerGroup = 4;                        // tiles a workgroup evaluates, a wave re-tests one
constexpr int kAlpha = kOrder + 1 + kOrder;              // coefficients and the zeros past them
constexpr int kWinWords = kWinX * kWinY / 2;             // two 16-bit counts a word

struct TileShared {
    double2 block[kAlpha];                               // alpha of the block's polynomial
    double2 tile[kTilesPerGroup][kAlpha];                // alpha of each tile's
    double2 patch[kTilesPerGroup * kPatches][kPatchOrder + 1];
    double patch_x[kTilesPerGroup * kPatches], patch_y[kTilesPerGroup * kPatches];   // centres
    double patch_inv[kTilesPerGroup * kPatches];         // 1 / radius
    unsigned win[2][kWinWords];                          // count windows, by turns
    int near_idx[kTilesPerGroup][kTileNear];
    int near_n[kTilesPerGroup];
    // of a tile with more near stars than that: which of the block's, 64 of its lists a word
    unsigned long long near_of[kTilesPerGroup][kBlockNear / 64];
};

// Image angle of lattice index base + off, base and off given as doubles:
// exactly image_angle's value (indices are below 2^53, so their sum is exact).
__device__ __forceinline__ double image_angle_at(double origin, double base, int off, double step) {
#pragma clang fp contract(off)
    double t = (base + (double)off) + 0.5;
    t = t * step;
    return origin + t;
}

// A lane's rays: a column in each of two neighbouring patches, kRows rows.
// (One patch at a time makes the stars' loads and loop 15 % slower; all four
// of a tile's row spill at three workgroups a compute unit.)
constexpr int kCols = 2;
constexpr int kRows = kPatchRays / 64;

// Star (sx, sy, sm) added to a lane's rays, one reciprocal for all eight: a
// product tree with the mass at its root, whose inverse is refined twice.  Of a
// star's term on its own rays the error is at most 11 units of 2^-53 (6 seen,
// RMS 1.6); one refinement leaves up to 19 (RMS 2.4), as does a reciprocal for
// each ray with one (RMS 2.1), which takes 16 % longer where a tile has about
// 300 near stars (60000 stars, 3000^2 rays: 873 us for 736).  A ray on the star
// turns all eight NaN (see expansion_tile_kernel).
__device__ __forceinline__ void near_star(double sx, double sy, double sm, const double (&tx)[kCols],
                                          const double (&ty)[kRows], double (&ax)[kCols][kRows],
                                          double (&ay)[kCols][kRows]) {
    double ey[kRows], ey2[kRows];
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        ey[k] = ty[k] - sy;
        ey2[k] = ey[k] * ey[k];
    }
    double ex[kCols], r2[kCols * kRows], w[kCols * kRows];
#pragma unroll
    for (int c = 0; c < kCols; ++c) {
        ex[c] = tx[c] - sx;
#pragma unroll
        for (int k = 0; k < kRows; ++k) r2[c * kRows + k] = __builtin_fma(ex[c], ex[c], ey2[k]);
    }
    fine_scaled_reciprocals<kCols * kRows>(r2, sm, w);
#pragma unroll
    for (int c = 0; c < kCols; ++c)
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            ax[c][k] = __builtin_fma(w[c * kRows + k], ex[c], ax[c][k]);
            ay[c][k] = __builtin_fma(w[c * kRows + k], ey[k], ay[c][k]);
        }
}

// Entry e of a block's near lists, one after the other; before[w] is the first
// entry of wave w's list.
__device__ __forceinline__ int block_near(const BlockFar *f, const int (&before)[kWaves], int e) {
    const int w = (e >= before[1]) + (e >= before[2]) + (e >= before[3]);
    return f->outer_idx[w][e - (w == 0 ? 0 : w == 1 ? before[1] : w == 2 ? before[2] : before[3])];
}

// The stars a tile sums directly, one after the other, uniform in the wave:
// all stars when the block's lists have overflowed, else the tile's near
// stars; body(x, y, m).  The next star's record is loaded while the current one
// is summed (all of 16602 stars, 74 x 370 rays: 6.15 ms for 6.88 without).
// Near stars come 64 at a time, indices in the lanes.  A tile's own list gives
// the indices without a trip to memory; one with more near stars than that
// takes the block's lists, of which near_of marks its own (40000 stars, 2000^2
// rays, blocks of 2 x 2 tiles of 257 near stars and more: 431 us a map, 1027
// when such a tile summed all of its block's).
template <class Body>
__device__ __forceinline__ void for_tile_direct(const TileShared &sh, int t, const ConstStar *st, const BlockFar *f,
                                                bool all, int n_stars, Body body) {
    if (all) {
        if (n_stars == 0) return;
        double sx = st[0].x, sy = st[0].y, sm = st[0].m;
        for (int k = 1; k <= n_stars; ++k) {
            asm volatile("" : "+s"(sx), "+s"(sy), "+s"(sm));   // as below
            const int next = k < n_stars ? k : 0;
            const double nx = st[next].x, ny = st[next].y, nm = st[next].m;
            __builtin_amdgcn_sched_barrier(0);
            body(sx, sy, sm);
            sx = nx;
            sy = ny;
            sm = nm;
        }
        return;
    }
    const int lane = threadIdx.x % 64, cnt = uniform(sh.near_n[t]);
    const bool own = cnt <= kTileNear;
    int before[kWaves] = {}, total = 0;
    if (!own)
        for (int w = 0; w < kWaves; ++w) {
            before[w] = total;
            total += uniform(f->outer_n[w]);
        }
    const int entries = own ? cnt : total;
    for (int i0 = 0; i0 < entries; i0 += 64) {   // uniform
        int idx = 0;
        unsigned long long left;   // which of the 64 are the tile's (uniform)
        if (own) {
            idx = sh.near_idx[t][i0 + lane];
            left = entries - i0 < 64 ? (1ull << (entries - i0)) - 1ull : ~0ull;
        } else {
            left = (unsigned long long)uniform64((int64_t)sh.near_of[t][i0 / 64]);
            if (i0 + lane < entries) idx = block_near(f, before, i0 + lane);
        }
        if (left == 0) continue;
        int k = __builtin_amdgcn_readlane(idx, __builtin_ctzll(left));
        double sx = st[k].x, sy = st[k].y, sm = st[k].m;
        while (left != 0) {
            asm volatile("" : "+s"(sx), "+s"(sy), "+s"(sm));   // the current record is here
            const unsigned long long rest = left & (left - 1);
            k = __builtin_amdgcn_readlane(idx, __builtin_ctzll(rest != 0 ? rest : left));
            const double nx = st[k].x, ny = st[k].y, nm = st[k].m;
            __builtin_amdgcn_sched_barrier(0);                 // the loads stay ahead of the sum
            body(sx, sy, sm);
            sx = nx;
            sy = ny;
            sm = nm;
            left = rest;
        }
    }
}

// The tiles of the blocks of L x L tiles, after the block pass.  Workgroup g
// takes kTilesPerGroup tiles of block g / kSubs (for L = 4 a row of them, for
// L = 2 the whole block, for L = 1 the one tile), in three phases:
//   1. One wave per tile re-centres the block's polynomial on its tile,
//      re-tests the block's near stars (far ones join the polynomial, near
//      ones go to the tile's list, and are marked in the block's) and sums the lanes' series.  A wave does
//      this alone, without a barrier: with the four waves sharing each tile's
//      stars, every wave still had to sum all 50 components, four times the
//      work, between two barriers a tile.
//   2. The tiles' polynomials are re-centred on their 16 patches of 16 x 16
//      rays, keeping kPatchOrder terms.  A patch is a quarter of its tile
//      across, so its terms fall four times as fast: a star farther than
//      rho / theta from the tile's centre is at least (1 / theta - 0.77) rho
//      from the patch's, whose radius is 0.239 rho, and what is dropped is below
//      (0.239 / (1 / theta - 0.77))^15 / (1 - 0.08) of its term: 1.1e-17
//      for theta = 0.25 and 3.8e-16 for 0.3, at or under the rounding of the
//      term.  One order less dropped 1.4e-16 and 4e-15: ten times the rounding
//      at 0.3 (the order takes 11 us of the 474 of 16384 stars, 8192^2 rays).
//      14 instead of 24 multiply-adds a ray.
//   3. Tile by tile, each wave evaluates four patches, four rays a lane: the
//      polynomial by Horner, the near stars directly, the pixel, the count.
//      Rays are counted as they come, in an LDS window around the pixel that
//      the tile's centre maps to without the near stars, two 16-bit counts a
//      word (a tile has 4096 rays); two windows take turns, so that a tile
//      needs one barrier, after which its window is merged into the map while
//      the next tile fills the other.
// Bound by VALU issue: about 167 instructions a ray (56 Horner, 8.6 per near
// star, 36 pixel and count, 15 for the first two phases), where 16 rays a lane
// at order 24 took 273: 16384 stars and 8192^2 rays 650 -> 425 us; the share
// of the chip's FP64 issue rate is alike.
// Three workgroups a compute unit: at four the registers spill.
// MAP: counts only, with pixel_coordinate's form of the division (the usual
// call); otherwise also the per-ray outputs, and the division where needed.
template <int L, int G, bool MAP>
__global__ __launch_bounds__(kThreads, 3) void expansion_tile_kernel(ShootParams p, double theta_open, int blocks_x,
                                                                     int skew, const BlockFar *__restrict__ far) {
    static_assert(G == 1 || (G == kTilesPerGroup && L > 1), "one tile or a group");
    constexpr int kSubs = L * L / G;
    __shared__ TileShared sh;
    const int lane = threadIdx.x % 64, wave = uniform(threadIdx.x / 64);
    const int pw = skew >= 0 ? 16 >> skew : 16 << -skew, ph = kPatchRays / pw;   // patch
    const int tw = kPatchSide * pw, th = kPatchSide * ph;                        // tile
    const int blk = (int)(blockIdx.x / kSubs), t_begin = (int)(blockIdx.x % kSubs) * G;
    const int64_t b_i = (int64_t)(blk % blocks_x) * (tw * L);
    const int64_t b_j = (int64_t)(blk / blocks_x) * (th * L);
    const ConstStar *st = const_stars(uniform_ptr(p.stars));
    const BlockFar *f = far + blk;
    const int n = uniform(p.n_stars);
    const double inv_theta = uniform_f64(1.0 / theta_open);

    bool overflow = false;
    int n_outer = 0, before[kWaves];   // the block's near stars, and those of earlier lists
    for (int w = 0; w < kWaves; ++w) {
        const int cnt = uniform(f->outer_n[w]);
        before[w] = n_outer;
        n_outer += cnt;
        overflow |= cnt > kNearPerWave;
    }
    for (int e = threadIdx.x; e < 2 * kWinWords; e += kThreads) sh.win[0][e] = 0;
    if (threadIdx.x < kAlpha) {
        double2 v = make_double2(0.0, 0.0);
        if (threadIdx.x <= kOrder) {
            const double fq = kFactorial.f[threadIdx.x];
            v = make_double2(f->A[threadIdx.x].x * fq, f->A[threadIdx.x].y * fq);
        }
        (L == 1 ? sh.tile[0] : sh.block)[threadIdx.x] = v;
    }
    __syncthreads();

    // --- phase 1
    if (L == 1) {
        // the block is the tile: its near stars, in one list, or every one of the block's
        if (threadIdx.x == 0) sh.near_n[0] = n_outer;
        if (!overflow && n_outer <= kTileNear)
            for (int w = 0; w < kWaves; ++w)
                for (int i = threadIdx.x; i < uniform(f->outer_n[w]); i += kThreads)
                    sh.near_idx[0][before[w] + i] = f->outer_idx[w][i];
        if (threadIdx.x < kBlockNear / 64) {
            const int in = n_outer - 64 * (int)threadIdx.x;   // entries of this word
            sh.near_of[0][threadIdx.x] = in >= 64 ? ~0ull : in > 0 ? (1ull << in) - 1ull : 0ull;
        }
    } else if (!overflow && wave < G) {
        const int t = t_begin + wave;
        double bcx, bcy, brho, cx, cy, rho;
        region_uniform(p, b_i, b_j, tw * L, th * L, bcx, bcy, brho);
        region_uniform(p, b_i + (int64_t)(t % L) * tw, b_j + (int64_t)(t / L) * th, tw, th, cx, cy, rho);
        const double r_near = rho * inv_theta, r_near2 = uniform_f64(r_near * r_near);
        double2 acc[kOrder + 1];
#pragma unroll
        for (int q = 0; q <= kOrder; ++q) acc[q] = make_double2(0.0, 0.0);
        int found = 0;   // near stars so far (uniform in the wave)
        for (int base = 0; base < n_outer; base += 64) {
            const int e = base + lane;
            bool near = false;
            int k = 0;
            if (e < n_outer) {
                k = block_near(f, before, e);
                const double sx = st[k].x, sy = st[k].y, sm = st[k].m;
                const double dx = cx - sx, dy = cy - sy;
                const double d2 = dx * dx + dy * dy;
                near = d2 <= r_near2;
                if (!near) {
                    const double inv = 1.0 / d2;
                    const double2 u = make_double2(dx * inv, -dy * inv);        // 1 / (c - z_k)
                    const double2 mu = make_double2(-u.x * rho, -u.y * rho);    // -u rho
                    double2 tq = make_double2(sm * u.x, sm * u.y);              // m u
#pragma unroll
                    for (int q = 0; q <= kOrder; ++q) {
                        acc[q].x += tq.x;
                        acc[q].y += tq.y;
                        if (q < kOrder) tq = cmul(tq, mu);
                    }
                }
            }
            const unsigned long long ball = __ballot(near);
            if (near) {
                const int pos = found + __popcll(ball & ((1ull << lane) - 1ull));
                if (pos < kTileNear) sh.near_idx[wave][pos] = k;
            }
            found += __popcll(ball);
            if (lane == 0) sh.near_of[wave][base / 64] = ball;
        }
        if (lane == 0) sh.near_n[wave] = found;
        const double v = wave_reduce_coeffs(acc);
        // the block's polynomial re-centred: lane r takes coefficient r
        const double inv_brho = 1.0 / brho;
        const double sx = (cx - bcx) * inv_brho, sy = (cy - bcy) * inv_brho;
        const int r = lane <= kOrder ? lane : kOrder;
        double2 S = sh.block[r + kOrder];
#pragma unroll 4
        for (int j = kOrder; j >= 1; --j)
            S = recentre_step(S, sh.block[r + j - 1], sx * kInverse.f[j], sy * kInverse.f[j]);
        const double br = int_pow(rho * inv_brho, r);
        if (lane < kAlpha) sh.tile[wave][lane] = lane <= kOrder ? make_double2(S.x * br, S.y * br) : make_double2(0.0, 0.0);
        // plus the re-tested far stars'
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the stores above, by other lanes
        __builtin_amdgcn_wave_barrier();
        if (lane < 2 * (kOrder + 1)) {
            double *d = reinterpret_cast<double *>(sh.tile[wave]);
            d[lane] += v * kFactorial.f[lane / 2];
        }
    }
    __syncthreads();

    // --- phase 2: lane = (tile, patch), the waves share the coefficients:
    // wave w takes r = w, w + 4, ... (with one tile, lane group i of 16 takes
    // r = w + 4 i)
    if (!overflow) {   // uniform
        constexpr int kEach = G == 1 ? 1 : (kPatchOrder + kWaves) / kWaves;
        const int pt = lane % kPatches, id = G == 1 ? pt : lane;
        const int g = G == 1 ? 0 : lane / kPatches, r0 = wave + (G == 1 ? kWaves * (lane / kPatches) : 0);
        const int t = t_begin + g;
        const int64_t ti = b_i + (int64_t)(t % L) * tw, tj = b_j + (int64_t)(t / L) * th;
        double cx, cy, rho, qx, qy, qrho;
        region(p, ti, tj, tw, th, cx, cy, rho);
        region(p, ti + (pt % kPatchSide) * pw, tj + (pt / kPatchSide) * ph, pw, ph, qx, qy, qrho);
        const double inv_rho = 1.0 / rho;
        const double sx = (qx - cx) * inv_rho, sy = (qy - cy) * inv_rho, b = qrho * inv_rho;
        double2 S[kEach];
        const double2 *alpha = sh.tile[g] + r0;
#pragma unroll
        for (int i = 0; i < kEach; ++i) S[i] = alpha[kOrder];   // the term j = kOrder - 4 i (zero unless r0 = 0)
        // coefficient r = r0 + 4 i has terms up to j = kOrder - r
        recentre_run<1, kEach>(S, alpha, sx, sy, kOrder, kOrder - kWaves + 1);
        recentre_run<2, kEach>(S, alpha, sx, sy, kOrder - kWaves, kOrder - 2 * kWaves + 1);
        recentre_run<3, kEach>(S, alpha, sx, sy, kOrder - 2 * kWaves, kOrder - 3 * kWaves + 1);
        recentre_run<4, kEach>(S, alpha, sx, sy, kOrder - 3 * kWaves, 1);
#pragma unroll
        for (int i = 0; i < kEach; ++i) {
            const int r = r0 + kWaves * i;
            if (r <= kPatchOrder) {
                const double c = int_pow(b, r) * kInverseFactorial.f[r];
                sh.patch[id][r] = make_double2(S[i].x * c, S[i].y * c);
            }
        }
        if (r0 == 0) {
            sh.patch_x[id] = qx;
            sh.patch_y[id] = qy;
            sh.patch_inv[id] = 1.0 / qrho;
        }
    }
    __syncthreads();

    // --- phase 3
    const int lx = lane & (pw - 1), ly = lane / pw, dj = 64 / pw;   // a lane's rays are dj rows apart
    int binned = 0;   // this lane's rays in the source window
    int turn = 0;     // of the windows: only tiles that are evaluated take one
    for (int g = 0; g < G; ++g) {   // uniform trip count
        const int t = t_begin + g;
        const int64_t tile_i = b_i + (int64_t)(t % L) * tw, tile_j = b_j + (int64_t)(t / L) * th;
        if (tile_i >= p.nx || tile_j >= p.ny) continue;   // uniform: no ray of this tile is in the lattice block
        const int left = uniform((int)(p.nx - tile_i < tw ? p.nx - tile_i : tw));
        const int down = uniform((int)(p.ny - tile_j < th ? p.ny - tile_j : th));
        const double base_i = uniform_f64((double)(p.i0 + tile_i)), base_j = uniform_f64((double)(p.j0 + tile_j));
        unsigned *win = sh.win[turn];
        turn ^= 1;
        // the window's corner, from the tile's centre (its own polynomial's first coefficient)
        int ox, oy;
        {
            double cx, cy, rho, mx, my, c0x = 0.0, c0y = 0.0;
            region_uniform(p, tile_i, tile_j, tw, th, cx, cy, rho);
            if (!overflow) {
                c0x = sh.tile[g][0].x;
                c0y = sh.tile[g][0].y;
            }
            macro_term(p, cx, cy, mx, my);
            const double u = (cx - (mx + c0x) - p.X0) * p.ipx, v = (cy - (my - c0y) - p.Y0) * p.ipy;
            ox = uniform((int)fmin(fmax(u, -1e9), 1e9)) - kWinX / 2;   // (NaN: -1e9)
            oy = uniform((int)fmin(fmax(v, -1e9), 1e9)) - kWinY / 2;
        }
        // the wave's row of patches: rows pj ... pj + ph - 1 of the tile
        const int pj = wave * ph;
#pragma unroll 1
        for (int q0 = 0; q0 < kPatchSide; q0 += kCols) {
            const int pi = q0 * pw, pid0 = g * kPatches + wave * kPatchSide + q0;
            if (pi >= left || pj >= down) continue;   // uniform
            double tx[kCols], ty[kRows], ax[kCols][kRows], ay[kCols][kRows];
#pragma unroll
            for (int c = 0; c < kCols; ++c) tx[c] = image_angle_at(p.x0, base_i, pi + c * pw + lx, p.dx);
#pragma unroll
            for (int k = 0; k < kRows; ++k) ty[k] = image_angle_at(p.y0, base_j, pj + ly + dj * k, p.dy);
#pragma unroll
            for (int c = 0; c < kCols; ++c) {
                // far field: Horner in s = (z - c) / rho; f = alpha_x - i alpha_y is
                // then added to the macro term
                double fx[kRows], fy[kRows];
                if (!overflow) {
                    const int pid = pid0 + c;
                    const double inv_rho = sh.patch_inv[pid], py = sh.patch_y[pid];
                    const double wx = (tx[c] - sh.patch_x[pid]) * inv_rho;
                    double wy[kRows];
                    const double2 top = sh.patch[pid][kPatchOrder];
#pragma unroll
                    for (int k = 0; k < kRows; ++k) {
                        wy[k] = (ty[k] - py) * inv_rho;
                        fx[k] = top.x;
                        fy[k] = top.y;
                    }
#pragma unroll
                    for (int r = kPatchOrder - 1; r >= 0; --r) {
                        const double2 b = sh.patch[pid][r];
#pragma unroll
                        for (int k = 0; k < kRows; ++k) {
                            const double hx = fx[k], hy = fy[k];
                            fx[k] = __builtin_fma(hx, wx, __builtin_fma(-hy, wy[k], b.x));
                            fy[k] = __builtin_fma(hx, wy[k], __builtin_fma(hy, wx, b.y));
                        }
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < kRows; ++k) fx[k] = fy[k] = 0.0;
                }
#pragma unroll
                for (int k = 0; k < kRows; ++k) {
                    double mx, my;
                    macro_term(p, tx[c], ty[k], mx, my);
                    ax[c][k] = mx + fx[k];
                    ay[c][k] = my - fy[k];
                }
            }
            for_tile_direct(sh, g, st, f, overflow, n,
                            [&](double sx, double sy, double sm) { near_star(sx, sy, sm, tx, ty, ax, ay); });
            bool bad = false;
#pragma unroll
            for (int c = 0; c < kCols; ++c)
#pragma unroll
                for (int k = 0; k < kRows; ++k) bad |= !__builtin_isfinite(ax[c][k] + ay[c][k]);
            if (__builtin_amdgcn_ballot_w64(bad) != 0) {   // uniform: a ray on a star, or far out of range
                // the rays with such sums again, one by one, a division a star;
                // through private arrays, so that this cold path takes no
                // registers of the rest
                double sum[2][kCols * kRows];
#pragma unroll
                for (int c = 0; c < kCols; ++c)
#pragma unroll
                    for (int k = 0; k < kRows; ++k) {
                        sum[0][c * kRows + k] = ax[c][k];
                        sum[1][c * kRows + k] = ay[c][k];
                    }
#pragma unroll 1
                for (int q = 0; q < kCols * kRows; ++q) {
                    const bool again = !__builtin_isfinite(sum[0][q]) || !__builtin_isfinite(sum[1][q]);
                    if (__builtin_amdgcn_ballot_w64(again) == 0) continue;   // uniform
                    const int c = q / kRows, k = q % kRows, pid = pid0 + c;
                    const double x = image_angle_at(p.x0, base_i, pi + c * pw + lx, p.dx);
                    const double y = image_angle_at(p.y0, base_j, pj + ly + dj * k, p.dy);
                    double fx = 0.0, fy = 0.0, mx, my;
                    if (!overflow) {
                        const double inv_rho = sh.patch_inv[pid];
                        const double wx = (x - sh.patch_x[pid]) * inv_rho, wy = (y - sh.patch_y[pid]) * inv_rho;
#pragma unroll 1
                        for (int r = kPatchOrder; r >= 0; --r) {
                            const double2 b = sh.patch[pid][r];
                            const double hx = fx, hy = fy;
                            fx = __builtin_fma(hx, wx, __builtin_fma(-hy, wy, b.x));
                            fy = __builtin_fma(hx, wy, __builtin_fma(hy, wx, b.y));
                        }
                    }
                    macro_term(p, x, y, mx, my);
                    double sxx = mx + fx, syy = my - fy;
                    for_tile_direct(sh, g, st, f, overflow, n, [&](double sx, double sy, double sm) {
                        const double ex = x - sx, ey = y - sy;
                        const double w = sm / __builtin_fma(ex, ex, ey * ey);
                        sxx = __builtin_fma(w, ex, sxx);
                        syy = __builtin_fma(w, ey, syy);
                    });
                    if (again) {
                        sum[0][q] = sxx;
                        sum[1][q] = syy;
                    }
                }
#pragma unroll
                for (int c = 0; c < kCols; ++c)
#pragma unroll
                    for (int k = 0; k < kRows; ++k) {
                        ax[c][k] = sum[0][c * kRows + k];
                        ay[c][k] = sum[1][c * kRows + k];
                    }
            }
            // Eq. (2), the pixel, the count
#pragma unroll
            for (int c = 0; c < kCols; ++c) {
                const int i = pi + c * pw + lx;
                int32_t is[kRows], js[kRows];
                {
#pragma clang fp contract(off)
                    if (MAP || p.fast_pixels) {   // uniform
#pragma unroll
                        for (int k = 0; k < kRows; ++k)
                            window_pixel(p, pixel_coordinate(tx[c] - ax[c][k], p.X0, p.Px, p.ipx),
                                         pixel_coordinate(ty[k] - ay[c][k], p.Y0, p.Py, p.ipy), is[k], js[k]);
                    } else {
#pragma unroll
                        for (int k = 0; k < kRows; ++k)
                            window_pixel(p, ((tx[c] - ax[c][k]) - p.X0) / p.Px, ((ty[k] - ay[c][k]) - p.Y0) / p.Py,
                                         is[k], js[k]);
                    }
                }
#pragma unroll
                for (int k = 0; k < kRows; ++k) {
                    const bool mine = i < left && pj + ly + dj * k < down;
                    if (!MAP && mine) {
                        const int64_t o = (tile_j + pj + ly + dj * k) * p.nx + tile_i + i;
                        if (p.beta_x) p.beta_x[o] = tx[c] - ax[c][k];
                        if (p.beta_y) p.beta_y[o] = ty[k] - ay[c][k];
                        if (p.bin) p.bin[o] = is[k] < 0 ? -1 : js[k] * p.NX + is[k];
                    }
                    if (!mine || (!MAP && !p.counts)) is[k] = -1;
                    const unsigned ux = (unsigned)(is[k] - ox), uy = (unsigned)(js[k] - oy);
                    const bool in = is[k] >= 0, in_win = ux < (unsigned)kWinX && uy < (unsigned)kWinY;
                    binned += in ? 1 : 0;
                    if (in && in_win) atomicAdd(&win[(uy * kWinX + ux) / 2], ux % 2 ? 0x10000u : 1u);
                    if (in && !in_win) atomicAdd(&p.counts[js[k] * p.NX + is[k]], 1);
                }
                __builtin_amdgcn_sched_barrier(0);   // keep the columns' temporaries apart
            }
        }
        if (!MAP && !p.counts) continue;   // uniform
        __syncthreads();   // the window is complete; the one before it has been merged
        // a wave per row of the window, 8 rows read ahead of their tests
        const int gx = ox + lane, half = lane % 2 * 16;
        const bool in_map = gx >= 0 && gx < p.NX;
#pragma unroll 1
        for (int r0 = 0; r0 < kWinY / kWaves; r0 += 8) {
            unsigned v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = win[(((r0 + u) * kWaves + wave) * kWinX + lane) / 2];
            if (__builtin_amdgcn_ballot_w64((v[0] | v[1] | v[2] | v[3] | v[4] | v[5] | v[6] | v[7]) != 0) == 0)
                continue;   // uniform: eight empty rows
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (v[u]) {
                    const int wy = (r0 + u) * kWaves + wave, gy = oy + wy;
                    win[(wy * kWinX + lane) / 2] = 0;
                    const int cnt = (int)(v[u] >> half & 0xFFFFu);
                    if (cnt && in_map && gy >= 0 && gy < p.NY) atomicAdd(&p.counts[gy * p.NX + gx], cnt);
                }
            }
        }
    }
    if (p.n_binned) {   // uniform
        const long long all = wave_sum((long long)binned);
        if (lane == 0 && all) atomicAdd(p.n_binned, (unsigned long long)all);
    }
}

// The block pass (with or without cells), then the tiles: kTilesPerGroup a
// workgroup when that leaves every compute unit four workgroups, else one
// (2048^2 rays: 58 us against 72).
template <int L>
hipError_t launch_level(const ShootParams &p, const StarCells &cells, double theta_open, const TileGrid &g,
                        BlockFar *far, hipStream_t s) {
    const int64_t bx = (g.tiles_x + L - 1) / L, by = (g.tiles_y + L - 1) / L;
    const int64_t groups = L > 1 ? bx * by * (L * L / kTilesPerGroup) : 0;
    const bool grouped = groups >= 4 * kComputeUnits;
    if (!grid_fits(grouped ? groups : bx * by * L * L, kThreads)) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)(bx * by));
    if (cells.ncx > 0)
        hipLaunchKernelGGL(expansion_block_kernel<true>, grid, dim3(kThreads), 0, s, p, cells, theta_open, (int)bx,
                           g.w * L, g.h * L, far);
    else
        hipLaunchKernelGGL(expansion_block_kernel<false>, grid, dim3(kThreads), 0, s, p, cells, theta_open, (int)bx,
                           g.w * L, g.h * L, far);
    const bool map = p.counts && p.fast_pixels && !p.beta_x && !p.beta_y && !p.bin;
    if constexpr (L > 1) {
        if (grouped) {
            if (map)
                hipLaunchKernelGGL((expansion_tile_kernel<L, kTilesPerGroup, true>), dim3((unsigned)groups),
                                   dim3(kThreads), 0, s, p, theta_open, (int)bx, g.skew, far);
            else
                hipLaunchKernelGGL((expansion_tile_kernel<L, kTilesPerGroup, false>), dim3((unsigned)groups),
                                   dim3(kThreads), 0, s, p, theta_open, (int)bx, g.skew, far);
            return hipGetLastError();
        }
    }
    const dim3 tiles((unsigned)(bx * by * L * L));
    if (map)
        hipLaunchKernelGGL((expansion_tile_kernel<L, 1, true>), tiles, dim3(kThreads), 0, s, p, theta_open, (int)bx,
                           g.skew, far);
    else
        hipLaunchKernelGGL((expansion_tile_kernel<L, 1, false>), tiles, dim3(kThreads), 0, s, p, theta_open, (int)bx,
                           g.skew, far);
    return hipGetLastError();
}

// Each star cell's scaled multipole expansion, one thread per cell, its
// stars in their sorted order.
__global__ __launch_bounds__(kThreads) void star_cell_multipole_kernel(const Star *__restrict__ sorted,
                                                                      const int32_t *__restrict__ start, int ncx,
                                                                      int ncy, double gx0, double gy0, double h,
                                                                      double rc, double2 *__restrict__ mult) {
    const int c = blockIdx.x * kThreads + threadIdx.x;
    if (c >= ncx * ncy) return;
    const double cx = gx0 + ((double)(c % ncx) + 0.5) * h;
    const double cy = gy0 + ((double)(c / ncx) + 0.5) * h;
    const double inv = 1.0 / rc;
    double2 acc[kOrder + 1];
#pragma unroll
    for (int q = 0; q <= kOrder; ++q) acc[q] = make_double2(0.0, 0.0);
    for (int i = start[c]; i < start[c + 1]; ++i) {
        const Star st = sorted[i];
        const double2 t = make_double2((st.x - cx) * inv, (st.y - cy) * inv);   // (z_k - z_c) / r_c
        double2 tp = make_double2(st.m, 0.0);
#pragma unroll
        for (int q = 0; q <= kOrder; ++q) {
            acc[q].x += tp.x;
            acc[q].y += tp.y;
            if (q < kOrder) tp = cmul(tp, t);
        }
    }
#pragma unroll
    for (int q = 0; q <= kOrder; ++q) mult[(size_t)c * (kOrder + 1) + q] = acc[q];
}

}  // namespace

int expansion_order() { return kOrder; }

// The block that minimises a simple cost model: a block costs about
// N* + 16384 L^2 star-equivalents (its pass over all stars, then L^2 tiles of
// Horner steps, near stars and binning), and blocks run in rounds of three
// per compute unit, a part-filled round counted in proportion.  Keeping the
// tiles' sum with the block also keeps large blocks away from lattices of few
// blocks, where dense star fields would overflow a large block's near-star
// lists (then its tiles sum every star directly).  The 16384 is of a tile
// kernel about 1.5 times slower than the present one, star cells are taken for
// N* stars, and the field's density is not looked at.  Measured, the choice
// against blocks 1, 2 and 4 (us): 16384 stars, 8192^2 rays 4 of 1930, 765, 474;
// 16384 and 4096^2 2 of 523, 250, 186; 5000 and 2000^2 1 of 102, 89, 101;
// 262144 and 4096^2 2 of 559, 245, 168.  Where the lists of the block it picks
// overflow it loses far more: 200000 stars and 6000^2 rays over the whole field
// take 1.8 s in blocks of 4 x 4 tiles and 2.4 ms in single ones
// (raysh_set_expansion_block).
int expansion_block(const TileGrid &g, int64_t n_stars, int n_cu) {
    const int64_t slots = 3 * (int64_t)(n_cu > 0 ? n_cu : 256);
    int best = 1;
    double best_cost = 0.0;
    for (int L : {1, 2, 4}) {
        const int64_t blocks = ((g.tiles_x + L - 1) / L) * ((g.tiles_y + L - 1) / L);
        const double rounds = std::max(1.0, (double)blocks / (double)slots);   // a part-filled round runs faster
        const double cost = rounds * ((double)n_stars + 16384.0 * L * L);
        if (L == 1 || cost < best_cost) {
            best = L;
            best_cost = cost;
        }
    }
    return best;
}

size_t expansion_workspace_bytes(const TileGrid &g, int block) {
    const int64_t blocks = ((g.tiles_x + block - 1) / block) * ((g.tiles_y + block - 1) / block);
    return (size_t)blocks * sizeof(BlockFar);
}

hipError_t launch_shoot_expansion(const ShootParams &p, const StarCells &cells, double theta_open, const TileGrid &g,
                                  int block, void *workspace, hipStream_t s) {
    BlockFar *far = static_cast<BlockFar *>(workspace);
    switch (block) {
        case 1: return launch_level<1>(p, cells, theta_open, g, far, s);
        case 2: return launch_level<2>(p, cells, theta_open, g, far, s);
        case 4: return launch_level<4>(p, cells, theta_open, g, far, s);
        default: return hipErrorInvalidValue;
    }
}

void free_star_cells(StarCellStore &c) {
    if (c.sorted) (void)hipFree(c.sorted);
    if (c.start) (void)hipFree(c.start);
    if (c.mult) (void)hipFree(c.mult);
    c = StarCellStore{};
}

// The cell side balances a block's two costs: the stars of its open cells,
// tested one by one (their number grows as side^2), against the
// translations of the other cells (whose number falls as 1/side^2, each
// about 6 times the work of one star's expansion).  Their sum is least
// near side^2 = area / (2 sqrt(N*)) for theta_open = 0.25 (262144 stars,
// 4096^2 rays: 446, 422, 459 and 488 us for 1, 2, 4 and 8 in place of the 2);
// the grid is then coarsened until it fits the workgroup's tables.
hipError_t build_star_cells(const Star *d_stars, int64_t n_stars, hipStream_t s, StarCellStore &out) {
    free_star_cells(out);
    if (n_stars < 2 || n_stars > kCellMaxStars) return hipSuccess;   // no cells
    std::vector<Star> host((size_t)n_stars);
    hipError_t e = hipMemcpyAsync(host.data(), d_stars, (size_t)n_stars * sizeof(Star), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return e;
    double x0 = host[0].x, x1 = host[0].x, y0 = host[0].y, y1 = host[0].y;
    for (const Star &st : host) {
        x0 = std::min(x0, st.x);
        x1 = std::max(x1, st.x);
        y0 = std::min(y0, st.y);
        y1 = std::max(y1, st.y);
    }
    const double w = x1 - x0, hgt = y1 - y0, big = std::max(w, hgt);
    if (!(big > 0.0)) return hipSuccess;   // every star at one point: no cells
    const double area = std::max(w * hgt, 1e-6 * big * big);
    double side = std::sqrt(area / (2.0 * std::sqrt((double)n_stars)));
    int ncx = 0, ncy = 0;
    for (;;) {
        ncx = (int)std::min(std::floor(w / side) + 1.0, 1e9);
        ncy = (int)std::min(std::floor(hgt / side) + 1.0, 1e9);
        if (ncx <= kCellMaxRows && ncy <= kCellMaxRows && (int64_t)ncx * ncy <= kCellMaxCells) break;
        side *= 1.25;
    }
    const int n_cells = ncx * ncy;
    // counting sort of the stars by cell, index order within a cell
    std::vector<int32_t> cell((size_t)n_stars), start((size_t)n_cells + 1, 0);
    for (int64_t k = 0; k < n_stars; ++k) {
        const int i = std::min((int)((host[k].x - x0) / side), ncx - 1);
        const int j = std::min((int)((host[k].y - y0) / side), ncy - 1);
        cell[k] = j * ncx + i;
        ++start[cell[k] + 1];
    }
    int32_t most = 0;
    for (int c = 0; c < n_cells; ++c) most = std::max(most, start[c + 1]);
    if (most > kCellMaxPerCell) return hipSuccess;   // one thread per cell would take too long: no cells
    for (int c = 0; c < n_cells; ++c) start[c + 1] += start[c];
    std::vector<Star> sorted((size_t)n_stars);
    {
        std::vector<int32_t> fill(start.begin(), start.end() - 1);
        for (int64_t k = 0; k < n_stars; ++k) {
            Star st = host[k];
            st.pad = __builtin_bit_cast(double, (long long)k);   // the star's index
            sorted[fill[cell[k]]++] = st;
        }
    }
    StarCellStore c;
    e = hipMalloc(&c.sorted, (size_t)n_stars * sizeof(Star));
    if (e == hipSuccess) e = hipMalloc(&c.start, ((size_t)n_cells + 1) * sizeof(int32_t));
    if (e == hipSuccess) e = hipMalloc(&c.mult, (size_t)n_cells * (kOrder + 1) * sizeof(double2));
    if (e == hipSuccess)
        e = hipMemcpyAsync(c.sorted, sorted.data(), (size_t)n_stars * sizeof(Star), hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
        e = hipMemcpyAsync(c.start, start.data(), ((size_t)n_cells + 1) * sizeof(int32_t), hipMemcpyHostToDevice,
                           s);
    // cells hold every star in the closed square of their cell (the last row
    // and column also the stars on the far edge): r_c is the half-diagonal,
    // enlarged for the rounding of the cell assignment
    const double rc = side * std::sqrt(0.5) * (1.0 + 1e-12);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(star_cell_multipole_kernel, dim3((unsigned)((n_cells + kThreads - 1) / kThreads)),
                           dim3(kThreads), 0, s, c.sorted, c.start, ncx, ncy, x0, y0, side, rc, c.mult);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipStreamSynchronize(s);   // the host tables are released on return
    if (e != hipSuccess) {
        (void)hipGetLastError();
        free_star_cells(c);
        return e;
    }
    c.view = StarCells{c.sorted, c.start, c.mult, x0, y0, side, rc, ncx, ncy};
    out = c;
    return hipSuccess;
}

}  // namespace raysh

// k_nlist.hip -- ordered neighbour list (Sec. 3.3 of the paper).
//
// Three builders, with the same rows for positions in the box: by tiles of
// cells staged in LDS (kind 0, the default; described where it stands), by
// blocks of cells (kind 1) and by lanes over global memory (kind 2, also the
// walk of the tiles that the first leaves, and the direct pass).
//
// Block builder: one 64-lane wavefront per Morton-aligned 2x2x2 block of cells.
// The block's cells have consecutive Morton ranks, so its particles (the i
// side) are one contiguous index range.  The union of their stencils is the
// 4x4x4 cells around the block (fewer where a side has only 3 cells); lane m
// takes union cell m, the cells are put in ascending rank (each lane counts
// the smaller ranks, then pushes its data to that lane with ds_permute) and
// their particle ranges concatenate into one strictly ascending candidate
// sequence, as the paper's sorted stencil does.  Lanes walk the candidates 64
// at a time; for every particle i of the block the wave ballots the distance
// test and a hit's slot in i's row is the row's running count plus the hits
// in lower lanes (mbcnt).  Rows are ascending and deterministic, no atomics.
//
// Distance test: separations in FP32 from the particles' offsets inside their
// cells plus whole-cell offsets in the block frame.  Outside a narrow band
// around r_list^2 the FP32 value decides; inside it the exact FP64 rule
// (minimum image, fma order) decides, so the rows equal the FP64 definition
// bit for bit.  Candidates two cells away from i fail the test (cells are
// wider than r_list).
//
// One pass writes every row into a fixed-width scratch slab and the row
// sizes; a scan makes the CSR offsets and a compaction copies the rows into
// the CSR list.  Rows that do not fit the slab width send the build through
// a second, direct pass instead (same walk, writing at the scanned offsets).
//
// Lane builder (while all ranks fit 27 bits): one lane per particle i.  The
// lane ranks i's 27 stencil cells, sorts them by rank with a fixed comparison
// network (Batcher's odd-even merge sort), and walks them in that order, each cell's particles in index order, so its row comes out
// ascending with no cross-lane work.  Lanes of a wave walk their own k-th
// stencil cells together; the distance test is the same FP32 pre-test with
// the same exact FP64 band rule.
#include <climits>
#include <cmath>

#include "dpd_launch.h"

namespace dpd {

namespace {

constexpr int kWavesPerBlock = kBlock / kWave;

__device__ __forceinline__ int32_t wrap_cell(int32_t c, int32_t n)
{
    c = c < 0 ? c + n : c;
    return c >= n ? c - n : c;
}

// index into the (batch-wide) rank table
__device__ __forceinline__ int32_t lin_cell(const KParams& kp, int32_t cx, int32_t cy, int32_t cz)
{
    return kp.c_off + cx + kp.nc[0] * (cy + kp.nc[1] * cz);
}

__device__ __forceinline__ float min_image32(float d, float L)
{
    const float h = 0.5f * L;
    d = d > h ? d - L : d;
    return d < -h ? d + L : d;
}

// exact FP64 neighbour rule for one pair (same operations as everywhere else)
__device__ __forceinline__ bool exact_hit(const KParams& kp, const double* __restrict__ x, int64_t N,
                                          int32_t i, int32_t j)
{
    const double dx = min_image(x[i] - x[j], kp.L[0], kp.halfL[0]);
    const double dy = min_image(x[N + i] - x[N + j], kp.L[1], kp.halfL[1]);
    const double dz = min_image(x[2 * N + i] - x[2 * N + j], kp.L[2], kp.halfL[2]);
    return dist2(dx, dy, dz) < kp.rl2;
}

// the direct pass's launch, which every build ends with, also says whether
// the list fits
__device__ __forceinline__ void capacity_check(const int32_t* __restrict__ offset, int32_t n, int64_t capacity,
                                               int32_t* __restrict__ status)
{
    if (status && blockIdx.x == 0 && threadIdx.x == 0 && (int64_t)offset[n] > capacity)
        atomicOr(status, 1 /* DPD_STATUS_NLIST_OVERFLOW */);
}

// kDirect = false: rows go to a fixed-width scratch slab (row i at
// slab[i * K]) and row sizes to offset[]; a scan and k_nlist_compact then
// produce the CSR list.  kDirect = true: the same walk writes straight into
// the CSR list (needs the scanned offsets); it only runs when some row did
// not fit its K slab slots.
template <bool kDirect>
__device__ __forceinline__ void nlist_block(const KParams& kp, int32_t blk, int32_t n,
                                            const double* __restrict__ x, const float* __restrict__ x32,
                                            const int32_t* __restrict__ cell_start,
                                            const int32_t* __restrict__ rank_tab, int32_t* __restrict__ offset,
                                            int32_t* __restrict__ index, int32_t* __restrict__ slab,
                                            int32_t slab_k, int32_t* __restrict__ flag)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t N = n;

    // ---- the block and its particle range ----
    int32_t bx, by, bz;
    morton_unrank(blk, kp.nb[0], kp.nb[1], kp.nb[2], kp.nbits_b, &bx, &by, &bz);
    const int32_t o[3] = {2 * bx, 2 * by, 2 * bz};                 // block origin (cells)
    int32_t vd[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) vd[d] = (kp.nc[d] - o[d] >= 2) ? 2 : 1;
    const int32_t nv = vd[0] * vd[1] * vd[2];
    const int32_t r0 = rank_tab[lin_cell(kp, o[0], o[1], o[2])];
    const int32_t i_lo = cell_start[r0], i_hi = cell_start[r0 + nv];
    if (i_lo == i_hi) return;

    // ---- union of the block's stencils: lane m < U owns union cell m ----
    int32_t ulo[3], ucnt[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        ulo[d] = o[d] - 1;
        ucnt[d] = vd[d] + 2;
        if (kp.small_dim[d] && ucnt[d] > kp.nc[d]) { ulo[d] = 0; ucnt[d] = kp.nc[d]; }
    }
    const int32_t U = ucnt[0] * ucnt[1] * ucnt[2];
    int32_t myrank = INT_MAX, mystart = 0, mylen = 0, myoff = 0;
    if (lane < U) {
        const int32_t ux = lane % ucnt[0], uy = (lane / ucnt[0]) % ucnt[1], uz = lane / (ucnt[0] * ucnt[1]);
        const int32_t fx = ulo[0] + ux, fy = ulo[1] + uy, fz = ulo[2] + uz;   // block-frame cell
        myrank = rank_tab[lin_cell(kp, wrap_cell(fx, kp.nc[0]), wrap_cell(fy, kp.nc[1]), wrap_cell(fz, kp.nc[2]))];
        mystart = cell_start[myrank];
        mylen = cell_start[myrank + 1] - mystart;
        // cell offset from the block origin, packed as three signed bytes
        myoff = ((fx - o[0]) & 0xFF) | (((fy - o[1]) & 0xFF) << 8) | (((fz - o[2]) & 0xFF) << 16);
    }
    int32_t pos = 0;
    for (int m = 0; m < U; ++m) pos += (__builtin_amdgcn_readlane(myrank, m) < myrank) ? 1 : 0;
    pos = lane < U ? pos : lane;                                    // idle lanes keep their slot
    const int32_t s_start = __builtin_amdgcn_ds_permute(pos * 4, mystart);
    const int32_t s_len = __builtin_amdgcn_ds_permute(pos * 4, mylen);
    const int32_t s_off = __builtin_amdgcn_ds_permute(pos * 4, myoff);
    int32_t s_incl = s_len;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int32_t t = __shfl_up(s_incl, d, kWave);
        if (lane >= d) s_incl += t;
    }
    const int32_t total = __builtin_amdgcn_readlane(s_incl, kWave - 1);

    const float4* __restrict__ xw = reinterpret_cast<const float4*>(x32);
    const float cl0 = kp.cell_len32[0], cl1 = kp.cell_len32[1], cl2 = kp.cell_len32[2];
    const bool wrap_any = kp.small_dim[0] | kp.small_dim[1] | kp.small_dim[2];

    for (int32_t ib = i_lo; ib < i_hi; ib += kWave) {            // i particles, 64 at a time
        const int32_t ie = (i_hi - ib) < kWave ? i_hi : ib + kWave;
        // lane li holds particle ib + li: in-cell offsets and its row count
        float wix = 0.f, wiy = 0.f, wiz = 0.f;
        int32_t run = 0;
        if (lane < ie - ib) {
            const float4 w = xw[ib + lane];
            wix = w.x; wiy = w.y; wiz = w.z;
            run = kDirect ? offset[ib + lane] : 0;
        }
        for (int32_t kb = 0; kb < total; kb += kWave) {           // candidates, 64 at a time
            const int32_t k = kb + lane;
            const bool valid = k < total;
            // sorted union cell holding candidate k: binary search on the prefix
            int32_t m = 0;
#pragma unroll
            for (int step = 32; step > 0; step >>= 1) {
                const int32_t probe = __shfl(s_incl, m + step - 1, kWave);
                m = (probe <= k) ? m + step : m;
            }
            m = m < kWave ? m : kWave - 1;
            const int32_t cs = __shfl(s_start, m, kWave);
            const int32_t cin = __shfl(s_incl, m, kWave);
            const int32_t cln = __shfl(s_len, m, kWave);
            const int32_t cof = __shfl(s_off, m, kWave);
            const int32_t j = valid ? cs + (k - (cin - cln)) : -1;
            const float4 wj = xw[valid ? j : 0];
            const float pjx = wj.x + (float)(int8_t)(cof & 0xFF) * cl0;
            const float pjy = wj.y + (float)(int8_t)((cof >> 8) & 0xFF) * cl1;
            const float pjz = wj.z + (float)(int8_t)((cof >> 16) & 0xFF) * cl2;
            // walk the block's cells in rank order; inside cell g the i
            // side sits at whole-cell offset delta_g from the block origin,
            // which is folded into the candidate positions once per cell
            int32_t g = -1, g_end = ib, code = -1;
            float qx = 0.f, qy = 0.f, qz = 0.f;
            for (int32_t i = ib; i < ie; ++i) {
                while (i >= g_end) {                               // next non-empty block cell
                    ++g;
                    do { ++code; } while (!((code & 1) < vd[0] && ((code >> 1) & 1) < vd[1] && (code >> 2) < vd[2]));
                    g_end = cell_start[r0 + g + 1];
                    qx = pjx - (float)(code & 1) * cl0;
                    qy = pjy - (float)((code >> 1) & 1) * cl1;
                    qz = pjz - (float)(code >> 2) * cl2;
                }
                const int li = i - ib;
                float dx = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wix), li)) - qx;
                float dy = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wiy), li)) - qy;
                float dz = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wiz), li)) - qz;
                if (wrap_any) {
                    dx = kp.small_dim[0] ? min_image32(dx, kp.L32[0]) : dx;
                    dy = kp.small_dim[1] ? min_image32(dy, kp.L32[1]) : dy;
                    dz = kp.small_dim[2] ? min_image32(dz, kp.L32[2]) : dz;
                }
                const float r2 = __fmaf_rn(dz, dz, __fmaf_rn(dy, dy, dx * dx));
                const bool cand = valid && j != i;
                bool hit = cand && r2 < kp.list_lo32;
                const bool amb = cand && !hit && r2 < kp.list_hi32;
                if (__ballot(amb)) {
                    if (amb) hit = exact_hit(kp, x, N, i, j);
                }
                const uint64_t mask = __ballot(hit);
                const int32_t base = __builtin_amdgcn_readlane(run, li);
                const int32_t at = base + lanes_below(mask);
                const int32_t cnt = (int32_t)__popcll(mask);
                if (kDirect) {
                    if (hit) index[at] = j;
                } else {
                    if (hit && at < slab_k) slab[(int64_t)i * slab_k + at] = j;
                    if (base + cnt > slab_k && lane == 0) atomicOr(flag, 1);
                }
                run = (lane == li) ? base + cnt : run;
            }
        }
        if (!kDirect && lane < ie - ib) offset[ib + lane] = run;
    }
}

// blk counts the 2x2x2 blocks of all systems of a batch in turn; kW waves
// per workgroup, one block per wave
template <bool kDirect, bool kB, int kW>
__global__ __launch_bounds__(kW * kWave) void k_nlist(KParams kp, BatchView bv, int32_t n_blocks, int32_t n,
                                                      const double* __restrict__ x, const float* __restrict__ x32,
                                                      const int32_t* __restrict__ cell_start,
                                                      const int32_t* __restrict__ rank_tab,
                                                      int32_t* __restrict__ offset, int32_t* __restrict__ index,
                                                      int64_t capacity, int32_t* __restrict__ slab, int32_t slab_k,
                                                      int32_t* __restrict__ flag, int32_t* __restrict__ status,
                                                      Gate gate)
{
    if (gated_off(gate)) return;
    if constexpr (kDirect) capacity_check(offset, n, capacity, status);
    const int32_t blk = xcd_logical_id(blockIdx.x, gridDim.x) * kW + threadIdx.x / kWave;
    if (blk >= n_blocks) return;
    if (kDirect && (*flag == 0 || (int64_t)offset[n] > capacity)) return;
    if constexpr (kB) {
        const int32_t sy = find_segment(bv.b_off, bv.n_sys, blk);
        nlist_block<kDirect>(bv.kps[sy], blk - bv.b_off[sy], n, x, x32, cell_start, rank_tab, offset, index, slab,
                             slab_k, flag);
    } else {
        nlist_block<kDirect>(kp, blk, n, x, x32, cell_start, rank_tab, offset, index, slab, slab_k, flag);
    }
}

// ---- lane-per-particle builder ----

constexpr SortNet kNet27 = make_sort_net(27);
static_assert(kNet27.count == 156, "27-key odd-even merge network");

template <bool kDirect>
__device__ __forceinline__ void nlist_lane(const KParams& kp, int32_t i, int32_t n, const double* __restrict__ x,
                                           const float* __restrict__ x32, const uint32_t* __restrict__ cell_xyz,
                                           const int32_t* __restrict__ cell_start,
                                           const int32_t* __restrict__ rank_tab, int32_t* __restrict__ offset,
                                           int32_t* __restrict__ index, int32_t* __restrict__ slab,
                                           int32_t slab_k, int32_t* __restrict__ flag)
{
    const int64_t N = n;
    const uint32_t me = cell_xyz[i];
    const int32_t cx = (int32_t)(me & 1023u), cy = (int32_t)((me >> 10) & 1023u), cz = (int32_t)(me >> 20);
    // stencil keys: rank << 5 | code, code = (dx+1) + 3 (dy+1) + 9 (dz+1)
    uint32_t key[27];
#pragma unroll
    for (int c = 0; c < 27; ++c) {
        const int dx = c % 3 - 1, dy = (c / 3) % 3 - 1, dz = c / 9 - 1;
        const int32_t r = rank_tab[lin_cell(kp, wrap_cell(cx + dx, kp.nc[0]), wrap_cell(cy + dy, kp.nc[1]),
                                            wrap_cell(cz + dz, kp.nc[2]))];
        key[c] = ((uint32_t)r << 5) | (uint32_t)c;
    }
#pragma unroll
    for (int c = 0; c < kNet27.count; ++c) {
        const uint32_t u = key[kNet27.a[c]], v = key[kNet27.b[c]];
        key[kNet27.a[c]] = u < v ? u : v;
        key[kNet27.b[c]] = u < v ? v : u;
    }
    const float4 wi = reinterpret_cast<const float4*>(x32)[i];
    const float4* __restrict__ xw = reinterpret_cast<const float4*>(x32);
    const float cl0 = kp.cell_len32[0], cl1 = kp.cell_len32[1], cl2 = kp.cell_len32[2];
    int32_t cnt = 0;
    int32_t* __restrict__ out = kDirect ? index + offset[i] : slab + (int64_t)i * slab_k;
    const int32_t cap = kDirect ? INT_MAX : slab_k;
    const bool coded = !kDirect && n <= kSlabJMask;
    // Loads run ahead of the tests: the next cell's bounds are requested when
    // a cell starts, candidates are tested two at a time while the two after
    // them are in flight, and a cell's first two are requested as the
    // previous cell ends.
    int32_t j0 = cell_start[key[0] >> 5], j1 = cell_start[(key[0] >> 5) + 1];
    float4 wa = xw[j0 < j1 ? j0 : i];
    float4 wb = xw[j0 + 1 < j1 ? j0 + 1 : i];
    auto test = [&](int32_t j, const float4& wj, float qx, float qy, float qz, uint32_t tagc) {
        const float dx = qx - wj.x, dy = qy - wj.y, dz = qz - wj.z;
        const float r2 = __fmaf_rn(dz, dz, __fmaf_rn(dy, dy, dx * dx));
        bool hit = j != i && r2 < kp.list_lo32;
        if (j != i && !hit && r2 < kp.list_hi32) hit = exact_hit(kp, x, N, i, j);
        if (hit) {
            if (cnt < cap) out[cnt] = (int32_t)((uint32_t)j | tagc);
            ++cnt;
        }
    };
#pragma unroll
    for (int q = 0; q < 27; ++q) {
        int32_t j0n = 0, j1n = 0;
        if (q + 1 < 27) {
            const int32_t rn = (int32_t)(key[q + 1] >> 5);
            j0n = cell_start[rn];
            j1n = cell_start[rn + 1];
        }
        const int c = (int)(key[q] & 31u);
        const uint32_t tagc = coded ? ((uint32_t)(c % 3) | ((uint32_t)((c / 3) % 3) << 2) |
                                       ((uint32_t)(c / 9) << 4)) << kSlabCodeShift
                                    : 0u;
        // i's cell-relative position minus the cell's whole-cell offset
        const float qx = wi.x - (float)(c % 3 - 1) * cl0;
        const float qy = wi.y - (float)((c / 3) % 3 - 1) * cl1;
        const float qz = wi.z - (float)(c / 9 - 1) * cl2;
        for (int32_t j = j0; j < j1; j += 2) {
            const float4 w0 = wa, w1 = wb;
            const bool two = j + 1 < j1;
            // the pair after this one inside the cell (clamped to its last
            // candidate; the next cell's first two are requested below)
            const int32_t last = j1 - 1;
            wa = xw[j + 2 < last ? j + 2 : last];
            wb = xw[j + 3 < last ? j + 3 : last];
            test(j, w0, qx, qy, qz, tagc);
            if (two) test(j + 1, w1, qx, qy, qz, tagc);
        }
        wa = xw[j0n < j1n ? j0n : i];
        wb = xw[j0n + 1 < j1n ? j0n + 1 : i];
        j0 = j0n;
        j1 = j1n;
    }
    if (!kDirect) {
        offset[i] = cnt;
        if (cnt > slab_k) atomicOr(flag, 1);
    }
}

// workgroups of the direct pass (a few per compute unit)
constexpr int32_t kDirectGrid = 2048;

template <bool kDirect, bool kB, int kW>
__global__ __launch_bounds__(kW * kWave) void k_nlist_lanes(KParams kp, BatchView bv, int32_t n,
                                                            const double* __restrict__ x,
                                                            const float* __restrict__ x32,
                                                            const uint32_t* __restrict__ cell_xyz,
                                                            const int32_t* __restrict__ cell_start,
                                                            const int32_t* __restrict__ rank_tab,
                                                            int32_t* __restrict__ offset,
                                                            int32_t* __restrict__ index, int64_t capacity,
                                                            int32_t* __restrict__ slab, int32_t slab_k,
                                                            int32_t* __restrict__ flag,
                                                            int32_t* __restrict__ status, Gate gate)
{
    if (gated_off(gate)) return;
    if constexpr (kDirect) capacity_check(offset, n, capacity, status);
    if (kDirect && (*flag == 0 || (int64_t)offset[n] > capacity)) return;
    // (the direct pass runs on a capped grid, each lane taking every
    // gridDim-th group of rows: it is launched for every build and returns
    // at once unless the slab overflowed)
    const int32_t g0 = xcd_logical_id(blockIdx.x, gridDim.x);
    for (int64_t b = g0; b * (kW * kWave) < n; b += kDirect ? gridDim.x : (int64_t)n) {
        const int32_t i = (int32_t)(b * (kW * kWave)) + (int32_t)threadIdx.x;
        if (i >= n) return;
        if constexpr (kB)
            nlist_lane<kDirect>(bv.kps[bv.sys_of[i]], i, n, x, x32, cell_xyz, cell_start, rank_tab, offset, index,
                                slab, slab_k, flag);
        else
            nlist_lane<kDirect>(kp, i, n, x, x32, cell_xyz, cell_start, rank_tab, offset, index, slab, slab_k,
                                flag);
    }
}

template <bool kDirect, int kW>
void launch_nlist_lanes(const KParams& kp, const BatchView& bv, int32_t n, const double* x, const float* x32,
                        const uint32_t* cell_xyz, const int32_t* cell_start, const int32_t* rank_tab,
                        int32_t* offset, int32_t* index, int64_t capacity, int32_t* slab, int32_t slab_k,
                        int32_t* flag, int32_t* status, hipStream_t s, Gate gate)
{
    const int32_t blocks = ceil_div(n, kW * kWave);
    const dim3 grid(kDirect && blocks > kDirectGrid ? kDirectGrid : blocks), block(kW * kWave);
    if (bv.kps)
        hipLaunchKernelGGL((k_nlist_lanes<kDirect, true, kW>), grid, block, 0, s, kp, bv, n, x, x32, cell_xyz,
                           cell_start, rank_tab, offset, index, capacity, slab, slab_k, flag, status, gate);
    else
        hipLaunchKernelGGL((k_nlist_lanes<kDirect, false, kW>), grid, block, 0, s, kp, bv, n, x, x32, cell_xyz,
                           cell_start, rank_tab, offset, index, capacity, slab, slab_k, flag, status, gate);
}

template <bool kDirect>
void launch_nlist_lanes(int waves, const KParams& kp, const BatchView& bv, int32_t n, const double* x,
                        const float* x32, const uint32_t* cell_xyz, const int32_t* cell_start,
                        const int32_t* rank_tab, int32_t* offset, int32_t* index, int64_t capacity,
                        int32_t* slab, int32_t slab_k, int32_t* flag, int32_t* status, hipStream_t s, Gate gate)
{
    if (waves == 1)
        launch_nlist_lanes<kDirect, 1>(kp, bv, n, x, x32, cell_xyz, cell_start, rank_tab, offset, index, capacity,
                                       slab, slab_k, flag, status, s, gate);
    else if (waves == 2)
        launch_nlist_lanes<kDirect, 2>(kp, bv, n, x, x32, cell_xyz, cell_start, rank_tab, offset, index, capacity,
                                       slab, slab_k, flag, status, s, gate);
    else
        launch_nlist_lanes<kDirect, 4>(kp, bv, n, x, x32, cell_xyz, cell_start, rank_tab, offset, index, capacity,
                                       slab, slab_k, flag, status, s, gate);
}

template <bool kDirect, int kW>
void launch_nlist_pass(const KParams& kp, const BatchView& bv, int32_t n_blocks, int32_t n, const double* x,
                       const float* x32, const int32_t* cell_start, const int32_t* rank_tab, int32_t* offset,
                       int32_t* index, int64_t capacity, int32_t* slab, int32_t slab_k, int32_t* flag,
                       int32_t* status, hipStream_t s, Gate gate)
{
    const dim3 grid(ceil_div(n_blocks, kW)), block(kW * kWave);
    if (bv.kps)
        hipLaunchKernelGGL((k_nlist<kDirect, true, kW>), grid, block, 0, s, kp, bv, n_blocks, n, x, x32, cell_start,
                           rank_tab, offset, index, capacity, slab, slab_k, flag, status, gate);
    else
        hipLaunchKernelGGL((k_nlist<kDirect, false, kW>), grid, block, 0, s, kp, bv, n_blocks, n, x, x32,
                           cell_start, rank_tab, offset, index, capacity, slab, slab_k, flag, status, gate);
}

template <bool kDirect>
void launch_nlist_pass(int waves, const KParams& kp, const BatchView& bv, int32_t n_blocks, int32_t n,
                       const double* x, const float* x32, const int32_t* cell_start, const int32_t* rank_tab,
                       int32_t* offset, int32_t* index, int64_t capacity, int32_t* slab, int32_t slab_k,
                       int32_t* flag, int32_t* status, hipStream_t s, Gate gate)
{
    if (waves == 1)
        launch_nlist_pass<kDirect, 1>(kp, bv, n_blocks, n, x, x32, cell_start, rank_tab, offset, index, capacity,
                                      slab, slab_k, flag, status, s, gate);
    else if (waves == 2)
        launch_nlist_pass<kDirect, 2>(kp, bv, n_blocks, n, x, x32, cell_start, rank_tab, offset, index, capacity,
                                      slab, slab_k, flag, status, s, gate);
    else
        launch_nlist_pass<kDirect, 4>(kp, bv, n_blocks, n, x, x32, cell_start, rank_tab, offset, index, capacity,
                                      slab, slab_k, flag, status, s, gate);
}

// ---- tile builder ----
//
// One workgroup per tile of kTileX x kTileY x kTileZ cells (consecutive
// Morton ranks, so the tile's particles are one index range).  The union of
// its cells' stencils, (kTileX+2) x (kTileY+2) x (kTileZ+2) cells, is staged
// in LDS: 16-bit positions and the particle indices, the cells in the order
// of kUnionOrder, which puts most cells that follow each other in rank side
// by side.  Each tile cell's 27 stencil cells are put in ascending rank once,
// by one lane, with the same sorting network; those that follow each other
// in LDS as well are joined, which leaves 10.5 runs of slots on average
// instead of 27; the runs are cut into steps of four candidates, 25 on
// average at density 3.  Each lane then walks its particle's steps in that
// order, so its row comes out ascending.  A step with a hit leaves one 16-bit
// word in LDS (first slot and four hit bits); the row is written from these
// words afterwards, two entries per store.
//
// Positions are counted in units of 1/13055 of the widest cell, 16 bits per
// component modulo five cells (a candidate's cell touches the particle's, so
// differences never wrap and squared distances stay below 2^31): four packed
// integer instructions give the squared distance less the list radius's,
// exact for the rounded positions, and its sign bit is the test.  Inside the
// band that their rounding leaves open the FP64 rule decides (0.01 candidates
// per particle at density 3).
//
// What bounds it: no one unit.  At 16M particles (density 3, seven waves per
// SIMD) a wave takes 2,665 vector instructions (33 per step of four candidates,
// 23 of them the distance test), one per 4.5 clocks and SIMD, 44 % of the issue
// peak; the LDS is busy 57 % of the time (21 % in bank conflicts), the address
// unit 44 %; the rest is waiting for LDS reads, barriers and the longest walk of
// each wave.  Time followed both the instructions and what is waited for: hence
// the wide steps, the joined runs and the integer test; a list of steps
// rather than of runs keeps the walk free of run ends (30 instructions per
// step fewer); rows leave two entries at a time since scattered stores cost
// the texture address unit a clock per lane (one at a time 1,482 us at 16M and
// 57 us at 262,144 particles of density 5, two 1,431 and 47, four 1,448 and
// 49).  Measured, the kernel before it and this one: 16M particles 1,660 and
// 1,440 us; 262,144 in a channel 51 and 45 us; 3,000 25 and 22 us.  Before,
// candidates were tested in FP32 cell by cell, two per step, 50 steps a row,
// and each stored or dropped by a scattered store of its own (2,783
// instructions a wave).
//
// In a grid narrower than the union (fewer than 10 x 6 x 6 cells) a cell can
// appear in the union at two places, as two periodic images, and is staged
// twice; every tile cell's 27 stencil cells are still distinct cells (3 or
// more per side), each at the image next to it, so no candidate is seen
// twice.  Tiles whose neighbourhood overflows the LDS, or holds a particle
// outside its cell, take the lane builder's walk over global memory.

constexpr int kTUX = kTileX + 2, kTUY = kTileY + 2, kTUZ = kTileZ + 2;
constexpr int kTU = kTUX * kTUY * kTUZ;          // union cells of a tile
constexpr int kTC = kTileX * kTileY * kTileZ;     // cells of a tile
// staged particles per tile: the workgroup's lanes (sized to the tile
// population's mean + 1.5 sigma) times 2.9, a little above the union's
// 360 / 128 cells per tile cell.  At density 3 (7 waves, 1,312 slots) the
// union's ~1,100 particles fluctuate by ~33, and the LDS use (39 KB) lets
// four workgroups share a compute unit.
template <int kW>
constexpr int tile_pos() { return (kW * kWave * 29 / 10 + 15) / 16 * 16; }
// union cell whose origin is the tile frame's origin (keeps |positions| small)
constexpr int kTFX = kTileX / 2 + 1, kTFY = kTileY / 2 + 1, kTFZ = kTileZ / 2 + 1;
// candidates a lane tests per step of the walk
constexpr int kCand = 4;
// steps of all tile cells together, each cell's followed by an empty one: the
// staged slots' share of a stencil, and a step for each of 8 runs that end
// inside one (a tile with more is left to the lane builder)
template <int kW>
constexpr int tile_steps() { return kTC * ((tile_pos<kW>() * 27 / kTU + kCand - 1) / kCand + 8); }
static_assert(tile_pos<16>() < 4096, "12-bit LDS slots in the runs, the steps and the words");

template <int kWords_, int kW>
struct TileLds {
    uint2 q[tile_pos<kW>() + kCand - 1];        // slots (see walk_pos); spare ones for reads past the end
    int32_t gl[kTU];                            // a union cell's first particle less its first slot
    uint32_t range[kTU];                        // its slots: start | end << 12
    uint32_t cstep[kTC];                        // steps of a tile cell: first | number << 16
    int32_t sum[2][kW];
    uint8_t off[28];                            // a stencil cell's place among the union cells
    uint32_t outside;                           // whether a particle is not in its cell
    alignas(16) uint16_t step[tile_steps<kW>()];            // first slot << 4 | four bits, the slots of the run
    alignas(16) uint16_t word[kWords_ * kW * kWave];
};
// words a lane keeps before it writes its hits out: what the LDS leaves when
// `groups` workgroups share a compute unit (rows have 14 words at most in 64
// lanes at density 3, 30 at 8)
template <int kW, int kGroups>
constexpr int tile_words()
{
    constexpr int lds = 160 * 1024 / kGroups / 64 * 64;
    constexpr int w = (lds - (int)sizeof(TileLds<0, kW>)) / (kW * kWave * 2);
    return w < 32 ? w : 32;
}

// The union cells in their order in LDS: the 27 blocks of cells that lie in
// one neighbouring tile each, the tile itself among them, and inside a block
// by Morton code.  Cells of a block therefore ascend in rank (but for tiles
// clipped at a high face, where fewer of them join).
struct UnionOrder {
    uint16_t u[kTU];
};
constexpr UnionOrder make_union_order()
{
    UnionOrder o{};
    uint32_t key[kTU] = {};
    for (int u = 0; u < kTU; ++u) {
        const int c[3] = {u % kTUX, (u / kTUX) % kTUY, u / (kTUX * kTUY)};
        const int side[3] = {kTileX, kTileY, kTileZ};
        uint32_t k = 0;
        for (int d = 0; d < 3; ++d) k = 3 * k + (c[d] == 0 ? 0 : c[d] == side[d] + 1 ? 2 : 1);
        for (int b = 3; b >= 0; --b)
            for (int d = 2; d >= 0; --d) k = 2 * k + (((c[d] + side[d] - 1) % side[d]) >> b & 1);
        key[u] = k;
    }
    for (int u = 0; u < kTU; ++u) {
        int at = 0;
        for (int v = 0; v < kTU; ++v) at += key[v] < key[u] ? 1 : 0;
        o.u[at] = (uint16_t)u;
    }
    return o;
}
__constant__ const UnionOrder kUnionOrder = make_union_order();

// Whether a particle is in its cell, to a thousandth of it.  One that is not
// (a position outside the box, binned into the nearest cell, or no number) may
// be further from others than the walk's units span: its tiles are left to the
// lane builder, which lists it by its geometry.
__device__ __forceinline__ bool in_cell(const KParams& P, const float4& w)
{
    const float c0 = P.cell_len32[0], c1 = P.cell_len32[1], c2 = P.cell_len32[2];
    return fabsf(w.x - 0.5f * c0) <= 0.501f * c0 && fabsf(w.y - 0.5f * c1) <= 0.501f * c1 &&
           fabsf(w.z - 0.5f * c2) <= 0.501f * c2;
}

// A slot: the position of a particle in its cell in the walk's units, x | y << 16
// and z, and in the high half of the second word its union cell (9 bits) with the
// low two bits of the cell's coordinates (6 bits, as in the slab's code).
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint2 walk_pos(const KParams& P, const float4& w, int32_t ux, int32_t uy, int32_t uz,
                                          uint32_t cell)
{
    const float c0 = P.cell_len32[0], c1 = P.cell_len32[1], c2 = P.cell_len32[2], inv = P.tile_inv;
    const int32_t x = (int32_t)__builtin_rintf((w.x + (float)(ux - kTFX) * c0) * inv),
                  y = (int32_t)__builtin_rintf((w.y + (float)(uy - kTFY) * c1) * inv),
                  z = (int32_t)__builtin_rintf((w.z + (float)(uz - kTFZ) * c2) * inv);
    return make_uint2(((uint32_t)x & 0xFFFFu) | ((uint32_t)y << 16), ((uint32_t)z & 0xFFFFu) | cell << 16);
}

// squared distance plus neg_lo
__device__ __forceinline__ int32_t walk_test(const uint2& a, const uint2& b, int32_t neg_lo)
{
    const i16x2 xy = __builtin_bit_cast(i16x2, a.x) - __builtin_bit_cast(i16x2, b.x);
    const int32_t z = (int16_t)(a.y - b.y);
    return __builtin_amdgcn_sdot2(xy, xy, z * z + neg_lo, false);
}

__device__ __forceinline__ int32_t wave_max(int32_t v)
{
#pragma unroll 1
    for (int d = kWave / 2; d > 0; d >>= 1) {
        const int32_t o = __shfl_xor(v, d, kWave);
        v = o > v ? o : v;
    }
    return __builtin_amdgcn_readfirstlane(v);
}

// exclusive prefix of v over the workgroup (kW waves); total gets the sum
template <int kW>
__device__ __forceinline__ int32_t tile_excl_scan(int32_t v, int32_t* s_w, int32_t& total)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    int32_t incl = v;
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        const int32_t t = __shfl_up(incl, d, kWave);
        if (lane >= d) incl += t;
    }
    if (lane == kWave - 1) s_w[w] = incl;
    __syncthreads();
    int32_t base = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < kW; ++k) {
        const int32_t sw = s_w[k];
        base += k < w ? sw : 0;
        tot += sw;
    }
    total = tot;
    return base + incl - v;
}

// The tile's system and cells: tile origin o (cells), its extent v (clipped
// at the high faces) and its particle range [i_lo, i_hi).
struct TileGeom {
    const KParams* P;
    int32_t o0, o1, o2, v0, v1, v2;
    int32_t i_lo, i_hi;
};

template <bool kB>
__device__ __forceinline__ TileGeom tile_geom(const KParams& kp, const BatchView& bv, int32_t tile,
                                              const int32_t* __restrict__ cell_start,
                                              const int32_t* __restrict__ rank_tab)
{
    TileGeom g;
    int32_t t_loc = tile;
    g.P = &kp;
    if constexpr (kB) {
        const int32_t sy = find_segment(bv.t_off, bv.n_sys, tile);
        g.P = &bv.kps[sy];
        t_loc = tile - bv.t_off[sy];
    }
    const KParams& P = *g.P;
    const int32_t tx = t_loc % P.nt[0], ty = (t_loc / P.nt[0]) % P.nt[1], tz = t_loc / (P.nt[0] * P.nt[1]);
    g.o0 = tx * kTileX; g.o1 = ty * kTileY; g.o2 = tz * kTileZ;
    g.v0 = min(kTileX, P.nc[0] - g.o0); g.v1 = min(kTileY, P.nc[1] - g.o1); g.v2 = min(kTileZ, P.nc[2] - g.o2);
    // the origin cell has the tile's smallest rank; its cells are the next v0 v1 v2 ranks
    const int32_t r0 = rank_tab[lin_cell(P, g.o0, g.o1, g.o2)];
    g.i_lo = cell_start[r0];
    g.i_hi = cell_start[r0 + g.v0 * g.v1 * g.v2];
    return g;
}

template <bool kB, int kW, int kGroups>
__global__ __launch_bounds__(kW * kWave) void k_nlist_tiles(KParams kp, BatchView bv, int32_t n_tiles, int32_t n,
                                                            const double* __restrict__ x,
                                                            const float* __restrict__ x32,
                                                            const uint32_t* __restrict__ cell_xyz,
                                                            const int32_t* __restrict__ cell_start,
                                                            const int32_t* __restrict__ rank_tab,
                                                            int32_t* __restrict__ offset,
                                                            int32_t* __restrict__ slab, int32_t slab_k,
                                                            int32_t* __restrict__ flag,
                                                            int32_t* __restrict__ rest, Gate gate)
{
    if (gated_off(gate)) return;
    constexpr int kThreads = kW * kWave;
    constexpr int kTilePos = tile_pos<kW>(), kSteps = tile_steps<kW>(), kWords = tile_words<kW, kGroups>();
    static_assert(kThreads >= kTU && kThreads > kTC, "one thread per union cell, and waves to stage beside the cells'");
    __shared__ TileLds<kWords, kW> lds;
    // before the walk, in the words: each tile cell's runs (first slot | the
    // cell's steps before it << 12 | length mod 4 << 30), their number before
    // and an end after them; in the steps: ranks of the union cells and union
    // cell of every slot
    constexpr int kRuns = 29;
    static_assert(kCand == 4, "a run's length mod 4 in two bits");
    uint16_t* const s_seg = lds.step + 2 * kTU;
    int32_t* const s_rank = reinterpret_cast<int32_t*>(lds.step);
    uint32_t* const s_run = reinterpret_cast<uint32_t*>(lds.word);
    static_assert(2 * kRuns * kTC <= kWords * kThreads, "the runs fit in the words");
    static_assert(2 * kTU + kTilePos <= kSteps, "the ranks and the staging map fit in the steps");

    const int32_t tile = xcd_logical_id(blockIdx.x, gridDim.x);
    if (tile >= n_tiles) return;
    const TileGeom g = tile_geom<kB>(kp, bv, tile, cell_start, rank_tab);
    if (g.i_lo == g.i_hi) return;
    const KParams& P = *g.P;
    const int tid = threadIdx.x;
    // (the tile's slab rows are addressed with 32-bit byte offsets)
    const bool fits = (int64_t)(g.i_hi - g.i_lo) * slab_k * 4 + 4 * kTilePos < INT32_MAX;

    if (tid < 27) lds.off[tid] = (uint8_t)(tid % 3 + kTUX * (tid / 3 % 3 + kTUY * (tid / 9)));
    if (tid == 27) lds.outside = 0u;

    // ---- union cells: thread t owns the t-th in LDS ----
    int32_t cnt = 0, u = 0;
    if (fits && tid < kTU) {
        u = kUnionOrder.u[tid];
        const int32_t ux = u % kTUX, uy = (u / kTUX) % kTUY, uz = u / (kTUX * kTUY);
        int32_t rank = INT_MAX, gs = 0;
        if (ux < g.v0 + 2 && uy < g.v1 + 2 && uz < g.v2 + 2) {
            rank = rank_tab[lin_cell(P, wrap_cell(g.o0 + ux - 1, P.nc[0]), wrap_cell(g.o1 + uy - 1, P.nc[1]),
                                     wrap_cell(g.o2 + uz - 1, P.nc[2]))];
            gs = cell_start[rank];
            cnt = cell_start[rank + 1] - gs;
        }
        s_rank[u] = rank;
        lds.gl[u] = gs;
    }
    int32_t total;
    const int32_t ls = tile_excl_scan<kW>(cnt, lds.sum[0], total);
    if (!fits || total > kTilePos) {
        // left to the lane builder's walk over global memory (k_nlist_tile_rest)
        if (tid == 0) rest[1 + atomicAdd(rest, 1)] = tile;
        return;
    }
    if (tid < kTU) {
        lds.gl[u] -= ls;
        lds.range[u] = (uint32_t)ls | (uint32_t)(ls + cnt) << 12;
        for (int32_t k = 0; k < cnt; ++k) s_seg[ls + k] = (uint16_t)u;
    }
    __syncthreads();

    // ---- staging: every union particle in the tile frame, by the waves that
    // have no cells below ----
    if (tid >= kTC) {
        constexpr int kStagers = kThreads - kTC, kRounds = (kTilePos + kStagers - 1) / kStagers;
        const float4* __restrict__ xw = reinterpret_cast<const float4*>(x32);
        // (all rounds' records requested before the first is converted)
        float4 w[kRounds];
        int32_t cell[kRounds];
#pragma unroll
        for (int q = 0; q < kRounds; ++q) {
            const int32_t p = tid - kTC + q * kStagers;
            cell[q] = 0;
            if (p < total) {
                cell[q] = s_seg[p];
                w[q] = xw[lds.gl[cell[q]] + p];
            }
        }
#pragma unroll
        for (int q = 0; q < kRounds; ++q) {
            const int32_t p = tid - kTC + q * kStagers, c = cell[q];
            const int32_t ux = c % kTUX, uy = (c / kTUX) % kTUY, uz = c / (kTUX * kTUY);
            const uint32_t code = (uint32_t)(ux & 3) | (uint32_t)(uy & 3) << 2 | (uint32_t)(uz & 3) << 4;
            if (p < total) {
                if (in_cell(P, w[q])) lds.q[p] = walk_pos(P, w[q], ux, uy, uz, (uint32_t)c | code << 9);
                else lds.outside = 1u;
            }
        }
    }

    // ---- each tile cell's runs: its non-empty stencil cells in ascending rank ----
    const bool is_cell = tid < kTC && tid % kTileX < g.v0 && (tid / kTileX) % kTileY < g.v1 &&
                         tid / (kTileX * kTileY) < g.v2;
    uint32_t key[27];
    uint32_t* const run = s_run + tid * kRuns;
    int32_t m = 0, n_run = 0;
    if (is_cell) {
        const int32_t u0 = tid % kTileX + kTUX * ((tid / kTileX) % kTileY + kTUY * (tid / (kTileX * kTileY)));
#pragma unroll
        for (int c = 0; c < 27; ++c)
            key[c] = ((uint32_t)s_rank[u0 + c % 3 + kTUX * ((c / 3) % 3 + kTUY * (c / 9))] << 5) | (uint32_t)c;
#pragma unroll
        for (int c = 0; c < kNet27.count; ++c) {
            const uint32_t a = key[kNet27.a[c]], b = key[kNet27.b[c]];
            key[kNet27.a[c]] = a < b ? a : b;
            key[kNet27.b[c]] = a < b ? b : a;
        }
#pragma unroll
        for (int q = 0; q < 27; ++q) key[q] = lds.range[u0 + lds.off[key[q] & 31u]];
        // Joined and counted without branches: a joined cell writes its run
        // again, with the new end, an empty one as it was; before the first
        // run stands one from 0 to ~0, which counts as no steps.
        uint32_t start = 0, end = ~0u;
#pragma unroll
        for (int q = 0; q < 27; ++q) {
            const uint32_t a = key[q] & 0xFFFu, b = key[q] >> 12;
            const bool some = a < b, turn = some && a != end;
            m += turn ? (int32_t)((end - start + kCand - 1) / kCand) : 0;
            start = turn ? a : start;
            n_run += turn ? 1 : 0;
            end = some ? b : end;
            run[n_run] = start | (uint32_t)m << 12 | (end - start) << 30;
        }
        m += (int32_t)((end - start + kCand - 1) / kCand);
        run[0] = (uint32_t)n_run;
        run[n_run + 1] = (uint32_t)m << 12;
        m += 1;                                                      // (the empty step)
    }
    int32_t n_steps;
    const int32_t at_step = tile_excl_scan<kW>(m, lds.sum[1], n_steps);
    if (n_steps > kSteps || lds.outside) {
        if (tid == 0) rest[1 + atomicAdd(rest, 1)] = tile;
        return;
    }
    if (is_cell) {
        lds.cstep[tid] = (uint32_t)at_step | (uint32_t)m << 16;
        lds.step[at_step + m - 1] = 0;
    } else if (tid < kTC) {
        run[0] = 0;
    }
    __syncthreads();

    // ---- the runs' steps: kPer lanes share a cell's runs ----
    constexpr int kPer = kThreads / kTC;
    if (tid < kPer * kTC) {
        const uint32_t* const cr = s_run + tid % kTC * kRuns;
        const int32_t nr = (int32_t)cr[0];
#pragma unroll 1
        for (int32_t r = 1 + tid / kTC; r <= nr; r += kPer) {
            const uint32_t w = cr[r], first = w >> 12 & 0x3FFFFu, rem = w >> 30;
            int32_t steps = (int32_t)((cr[r + 1] >> 12 & 0x3FFFFu) - first);
            uint16_t* st = lds.step + (lds.cstep[tid % kTC] & 0xFFFFu) + first;
            uint32_t word = w << kCand | 15u;
            for (; steps > 1; --steps, word += kCand << kCand) *st++ = (uint16_t)word;
            *st = (uint16_t)(rem ? word & ~15u | ((1u << rem) - 1u) : word);
        }
    }
    __syncthreads();

    // ---- the walk: one lane per particle of the tile ----
    // The next step's candidates and the step after the next are requested
    // from LDS before the current ones are tested.  A lane that has ended
    // stays on its empty step.
    const int32_t neg_lo = -(int32_t)P.tile_lo;
    const uint32_t band = P.tile_band;
    const int64_t N = n;
    // The tile's slab rows through a buffer resource: a row longer than the
    // slab width runs on into the next rows of the tile (stores past the
    // tile's last row are dropped by the range check); such a row sets the
    // flag, and the whole slab is then discarded for the direct pass.
    const int32_t n_here = g.i_hi - g.i_lo;
    const auto rows = __builtin_amdgcn_make_buffer_rsrc(slab + (int64_t)g.i_lo * slab_k, (short)0,
                                                        n_here * slab_k * (int32_t)sizeof(int32_t), 0x00020000);
    const uint32_t code_bits = n <= kSlabJMask ? ~0u << kSlabCodeShift : 0u;      // none: uncoded slab
    // A hit's entry is its particle with the code the difference of the cell
    // coordinates plus one, each two bits wide: a subtraction without borrows
    // between them (the code's high bits set before and put right after).
    const uint32_t hbit = 0xA8000000u & code_bits;
    static_assert(0x2Au << kSlabCodeShift == 0xA8000000u && kSlabCodeShift == 26, "the code's high bits");
    uint16_t* const list = lds.word + tid;
    for (int32_t i = g.i_lo + tid; i < g.i_hi; i += kThreads) {
        const uint32_t me = cell_xyz[i];
        const int32_t lx = (int32_t)(me & 1023u) - g.o0, ly = (int32_t)((me >> 10) & 1023u) - g.o1,
                      lz = (int32_t)(me >> 20) - g.o2;
        const int32_t self = i - lds.gl[(lx + 1) + kTUX * ((ly + 1) + kTUY * (lz + 1))];
        const uint2 qi = lds.q[self];
        const uint32_t cs = lds.cstep[lx + kTileX * (ly + kTileY * lz)];
        // (one step or more: i's own cell is in its stencil)
        const int32_t n_st = (int32_t)(cs >> 16) - 1;
        const uint16_t* p = lds.step + (cs & 0xFFFFu);
        const uint16_t* const p_end = p + n_st;
        int32_t left = wave_max(n_st);
        const uint32_t own = (uint32_t)(lx & 3) << 26 | (uint32_t)(ly & 3) << 28 | (uint32_t)(lz & 3) << 30;
        const uint32_t own_lo = own & code_bits & ~hbit, own_hi = ~own & hbit;
        const int32_t row0 = (i - g.i_lo) * slab_k * (int32_t)sizeof(int32_t);
        int32_t rb = row0;                                // byte offset of the row's next entry
        uint32_t last = 0;                                // the one before, stored with the next in one store
        int32_t at = 0;
        auto next_step = [&] {
            p = p + 1 < p_end ? p + 1 : p_end;
            return (uint32_t)*p;
        };
        auto request = [&](uint32_t st, uint2 (&w)[kCand]) {
            const uint2* q = lds.q + (st >> kCand);
#pragma unroll
            for (int c = 0; c < kCand; ++c) w[c] = q[c];
        };
        // step st on the candidates w; the next step's are requested first
        auto step = [&](uint32_t& st, uint32_t st_n, const uint2 (&w)[kCand], uint2 (&w_n)[kCand]) {
            const uint32_t now = st;
            request(st_n, w_n);
            st = next_step();
            int32_t t[kCand];
            uint32_t hits = 0, open = ~0u;
#pragma unroll
            for (int c = kCand - 1; c >= 0; --c) {
                t[c] = walk_test(qi, w[c], neg_lo);
                hits = __builtin_amdgcn_alignbit(hits, (uint32_t)t[c], 31);      // hits << 1 | t < 0
                open = min(open, (uint32_t)t[c]);                 // below `band`: the FP64 rule decides
            }
            // rare: the wave branches on the ballot
            if (__builtin_expect(__ballot(open < band) != 0ull, 0)) {
#pragma unroll 1
                for (int c = 0; c < kCand; ++c) {
                    const int32_t q = c == 0 ? t[0] : c == 1 ? t[1] : c == 2 ? t[2] : t[3];
                    if ((now >> c & 1u) && (uint32_t)q < band) {
                        const int32_t sl = (int32_t)(now >> kCand) + c;
                        const int32_t j = lds.gl[lds.q[sl].y >> 16 & 511u] + sl;
                        if (exact_hit(P, x, N, i, j)) hits |= 1u << c;
                    }
                }
            }
            // written at the list's end, which moves past it if it holds a hit
            hits &= now;
            list[at] = (uint16_t)((now & ~15u) | hits);
            at += hits ? kThreads : 0;
        };
        uint32_t sa = *p, sb = next_step();
        uint2 wa[kCand], wb[kCand];
        request(sa, wa);
        while (left > 0) {
            do {
                step(sa, sb, wa, wb);
                step(sb, sa, wb, wa);
                left -= 2;
            } while (left > 0 && __ballot(at > (kWords - 4) * kThreads) == 0ull);
            // The words' hits, lowest bit first.  Reads run ahead: the word
            // after the current one, and a hit's union cell, used a turn later
            // (the particle itself stands for no hit).
            int32_t gp = 0, sl_p = self;
            uint32_t word = list[0], word_n = list[kThreads], cell_p = 0;
            for (bool more = true; more;) {
                more = __ballot(gp < at) != 0ull;
                int32_t sl = self;
                uint32_t cell = 0;
                if (gp < at) {
                    sl = (int32_t)(word >> kCand) + __builtin_ctz(word);
                    cell = lds.q[sl].y;
                    word &= word - 1u;                    // (its lowest set bit: one of the four)
                    const bool turn = (word & 15u) == 0u;
                    word = turn ? word_n : word;
                    gp += turn ? kThreads : 0;
                    word_n = list[gp + kThreads];
                }
                if (sl_p != self) {
                    const uint32_t e = (uint32_t)(lds.gl[cell_p >> 16 & 511u] + sl_p) | (cell_p << 1 & code_bits);
                    const uint32_t entry = ((e | hbit) - own_lo) ^ ((e ^ own_hi) & hbit);
                    rb += (int32_t)sizeof(int32_t);
                    if ((rb & 4) == 0) {
                        const i32x2 v = {(int32_t)last, (int32_t)entry};
                        __builtin_amdgcn_raw_buffer_store_b64(v, rows, rb - 8, 0, 0);
                    }
                    last = entry;
                }
                sl_p = sl;
                cell_p = cell;
            }
            at = 0;
        }
        if (rb & 4) __builtin_amdgcn_raw_buffer_store_b32((int32_t)last, rows, rb - 4, 0, 0);
        const int32_t row = (rb - row0) / (int32_t)sizeof(int32_t);
        offset[i] = row;
        if (row > slab_k) atomicOr(flag, 1);
    }
}

// Tiles the tile builder left (neighbourhood over the LDS capacity, or with a
// particle outside its cell): rest[0] tiles listed in rest[1..], their particles walked by the lane
// builder.  A lane's walk is one serial chain of some 60 us, and the tiles are
// few: one wave per workgroup, kRestParts of them to a tile, so that each
// lane walks one row (256 systems, of which the smallest leave some tiles:
// 125 us with a tile to a workgroup of four waves, in two rounds, 89 us now).
constexpr int kRestParts = 8;

template <bool kB>
__global__ __launch_bounds__(kWave) void k_nlist_tile_rest(KParams kp, BatchView bv, int32_t n,
                                                            const double* __restrict__ x,
                                                            const float* __restrict__ x32,
                                                            const uint32_t* __restrict__ cell_xyz,
                                                            const int32_t* __restrict__ cell_start,
                                                            const int32_t* __restrict__ rank_tab,
                                                            int32_t* __restrict__ offset,
                                                            int32_t* __restrict__ slab, int32_t slab_k,
                                                            int32_t* __restrict__ flag,
                                                            const int32_t* __restrict__ rest, Gate gate)
{
    if (gated_off(gate)) return;
    const int64_t count = (int64_t)rest[0] * kRestParts;
    for (int64_t t = blockIdx.x; t < count; t += gridDim.x) {
        const TileGeom g = tile_geom<kB>(kp, bv, rest[1 + t / kRestParts], cell_start, rank_tab);
        const int32_t first = g.i_lo + (int32_t)(t % kRestParts) * kWave;
        for (int32_t i = first + (int32_t)threadIdx.x; i < g.i_hi; i += kRestParts * kWave)
            nlist_lane<false>(*g.P, i, n, x, x32, cell_xyz, cell_start, rank_tab, offset, nullptr, slab, slab_k,
                              flag);
    }
}

template <bool kB, int kW, int kGroups>
void launch_nlist_tiles_t(const KParams& kp, const BatchView& bv, int32_t n_tiles, int32_t n, const double* x,
                          const float* x32, const uint32_t* cell_xyz, const int32_t* cell_start,
                          const int32_t* rank_tab, int32_t* offset, int32_t* slab, int32_t slab_k, int32_t* flag,
                          int32_t* rest, hipStream_t s, Gate gate)
{
    hipLaunchKernelGGL((k_nlist_tiles<kB, kW, kGroups>), dim3(n_tiles), dim3(kW * kWave), 0, s, kp, bv, n_tiles, n, x, x32,
                       cell_xyz, cell_start, rank_tab, offset, slab, slab_k, flag, rest, gate);
}

// tile pass, then the pass over the tiles it left; rest[0] must be 0
template <bool kB>
void launch_nlist_tiles(int waves, const KParams& kp, const BatchView& bv, int32_t n_tiles, int32_t n,
                        const double* x, const float* x32, const uint32_t* cell_xyz, const int32_t* cell_start,
                        const int32_t* rank_tab, int32_t* offset, int32_t* slab, int32_t slab_k, int32_t* flag,
                        int32_t* rest, hipStream_t s, Gate gate)
{
    // Workgroups sharing a compute unit: as many as its 32 waves allow, but four
    // of 6 waves (a fifth would leave the runs no room in the words) and one of 16
    // waves where each of the 256 units gets two tiles at most.  As many, and one
    // less with more words a lane, on 2M particles: 6 waves (density 2.4) 222 and
    // 257 us, 7 waves (3) 207 and 221, 10 waves (4.2) 267 and 327, 12 waves (5.2)
    // 270 and 363; 8 waves, the 256 systems, 444 and 561 us.  On 256 to 500 tiles
    // the order is the same or within 1.5 us (10 waves, 256 tiles: 35.0 and 33.6;
    // 12 waves, 405 tiles: 50 and 61).  16 waves, two and one with 32 words a lane
    // against 18: 10 systems of 4,608 particles, 180 tiles, 54.4 and 46.6 us; 1M
    // particles at r_c + skin, 1,200 tiles, 85 and 84 us, and 16 us more per build
    // in a long run with one.
#define DPD_TILE_CASE(W, G)                                                                                      \
    launch_nlist_tiles_t<kB, W, G>(kp, bv, n_tiles, n, x, x32, cell_xyz, cell_start, rank_tab, offset, slab,      \
                                   slab_k, flag, rest, s, gate)
    if (waves <= 6) DPD_TILE_CASE(6, 4);
    else if (waves <= 7) DPD_TILE_CASE(7, 4);
    else if (waves <= 8) DPD_TILE_CASE(8, 4);
    else if (waves <= 10) DPD_TILE_CASE(10, 3);
    else if (waves <= 12) DPD_TILE_CASE(12, 2);
    else if (n_tiles > 512) DPD_TILE_CASE(16, 2);
    else DPD_TILE_CASE(16, 1);
#undef DPD_TILE_CASE
    const int grid = n_tiles < 512 ? n_tiles * kRestParts : 512 * kRestParts;
    hipLaunchKernelGGL((k_nlist_tile_rest<kB>), dim3(grid), dim3(kWave), 0, s, kp, bv, n, x, x32, cell_xyz,
                       cell_start, rank_tab, offset, slab, slab_k, flag, (const int32_t*)rest, gate);
}

}  // namespace

// Waves per tile workgroup: the mean particle count of a tile plus 1.5
// standard deviations (a tile with more particles walks the rest in a
// second round), at least enough threads for one per union cell.
int nlist_tile_waves(int32_t n, int32_t n_cells)
{
    const double mean = (double)kTC * (double)n / (double)(n_cells > 0 ? n_cells : 1);
    const double need = mean + 1.5 * std::sqrt(mean);
    int w = (int)std::ceil(need / kWave);
    constexpr int kMinW = (kTU + kWave - 1) / kWave;
    return w < kMinW ? kMinW : (w > 16 ? 16 : w);
}

namespace {

// CSR list from the slab: one wave per 64 consecutive rows writes their
// entries [offset[i0], offset[i0 + 64]) in order, one entry per lane.
__global__ __launch_bounds__(kBlock) void k_nlist_compact(int32_t n, const int32_t* __restrict__ offset,
                                                          int64_t capacity, const int32_t* __restrict__ slab,
                                                          int32_t slab_k, const int32_t* __restrict__ flag,
                                                          int32_t* __restrict__ index)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t i0 = ((int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / kWave) * kWave;
    const int32_t mask = n <= kSlabJMask ? kSlabJMask : -1;      // strips coded stencil offsets
    if (i0 >= n || *flag != 0 || (int64_t)offset[n] > capacity) return;
    const int32_t ni = n - i0 < kWave ? (int32_t)(n - i0) : kWave;
    const int32_t own = (int32_t)i0 + (lane < ni ? lane : ni - 1);
    const int32_t e0 = offset[i0], e1 = offset[i0 + ni];
    int32_t rend = offset[own + 1];
    const int32_t prev = __shfl_up(rend, 1, kWave);
    int32_t rstart = lane == 0 ? e0 : prev;
    if (lane >= ni) { rstart = e1; rend = e1; }
    for (int32_t eb = e0; eb < e1; eb += kWave) {
        // rows ra..rb-1 overlap this batch; walk their ends with readlane
        const int32_t e = eb + lane;
        const int32_t ra = (int32_t)__popcll(__ballot(lane < ni && rend <= eb));
        const int32_t rb = (int32_t)__popcll(__ballot(lane < ni && rstart < eb + kWave));
        int32_t r = ra;
        int32_t rs = __builtin_amdgcn_readlane(rstart, ra < kWave ? ra : kWave - 1);
        for (int32_t q = ra; q < rb; ++q) {
            const int32_t t = __builtin_amdgcn_readlane(rend, q);
            if (e >= t) { r = q + 1; rs = t; }
        }
        if (e < e1) index[e] = slab[(i0 + r) * slab_k + (e - rs)] & mask;
    }
}

}  // namespace

// Slots per row of the scratch slab: about 2.5 times the mean neighbour
// count plus a margin (rows that do not fit fall back to the direct pass).
int32_t nlist_slab_width(double density, double rl2)
{
    const double mean = 4.18879020478639 * density * rl2 * sqrt(rl2);
    int32_t k = (int32_t)(2.5 * mean + 24.0);
    k = k < 48 ? 48 : k;
    return (k + 15) / 16 * 16;
}

// The tile and lane builders pack a rank and a 5-bit stencil code into 32
// bits; beyond 2^27 cells the block builder takes over.
static bool ranks_fit(const uint32_t* cell_xyz, int32_t n_cells)
{
    return cell_xyz && n_cells < (1 << 27);
}

bool nlist_slab_coded(int kind, const uint32_t* cell_xyz, int32_t n_cells, int32_t n)
{
    return (kind == 0 || kind == 2) && ranks_fit(cell_xyz, n_cells) && n <= kSlabJMask;
}

hipError_t launch_nlist(const KParams& kp, const BatchView& bv, int32_t n_cells, int32_t n_blocks, int32_t n_tiles,
                        int32_t n, const double* x, const float* x32, const uint32_t* cell_xyz,
                        const int32_t* cell_start, const int32_t* rank_tab, int32_t* offset, int32_t* index,
                        int64_t capacity, int32_t* slab, int32_t slab_k, int32_t* flag, int32_t* tile_rest,
                        int32_t* status, int32_t* scan_part, int waves, int kind, bool compact, hipStream_t s,
                        Gate gate, bool cleared)
{
    if (n <= 0) return hipSuccess;
    hipError_t e;
    const bool tiles = kind == 0 && ranks_fit(cell_xyz, n_cells);
    const bool lanes = tiles || (kind == 2 && ranks_fit(cell_xyz, n_cells));
    if (!cleared && (e = launch_zero3(offset + n, flag, tiles ? tile_rest : nullptr, s, gate)) != hipSuccess) return e;
    if (tiles) {
        const int tw = nlist_tile_waves(n, n_cells);
        if (bv.kps)
            launch_nlist_tiles<true>(tw, kp, bv, n_tiles, n, x, x32, cell_xyz, cell_start, rank_tab, offset, slab,
                                     slab_k, flag, tile_rest, s, gate);
        else
            launch_nlist_tiles<false>(tw, kp, bv, n_tiles, n, x, x32, cell_xyz, cell_start, rank_tab, offset, slab,
                                      slab_k, flag, tile_rest, s, gate);
    } else if (lanes)
        launch_nlist_lanes<false>(waves, kp, bv, n, x, x32, cell_xyz, cell_start, rank_tab, offset, index, capacity,
                                  slab, slab_k, flag, status, s, gate);
    else
        launch_nlist_pass<false>(waves, kp, bv, n_blocks, n, x, x32, cell_start, rank_tab, offset, index, capacity,
                                 slab, slab_k, flag, status, s, gate);
    if ((e = launch_scan(offset, (int64_t)n + 1, scan_part, s, gate)) != hipSuccess) return e;
    // without compaction the CSR index is left unwritten unless a row
    // overflowed the slab (then the direct pass below writes it).  The
    // compaction takes no gate: after a step that kept the last build's
    // rows it copies those rows again.
    if (compact)
        hipLaunchKernelGGL(k_nlist_compact, dim3(ceil_div(ceil_div(n, kWave), kWavesPerBlock)), dim3(kBlock), 0,
                           s, n, (const int32_t*)offset, capacity, (const int32_t*)slab, slab_k,
                           (const int32_t*)flag, index);
    // the capacity check, and rows that overflowed the slab: the lane builder's
    // walk writes the CSR rows directly (the same rows as the tile builder's)
    if (lanes)
        launch_nlist_lanes<true>(waves, kp, bv, n, x, x32, cell_xyz, cell_start, rank_tab, offset, index, capacity,
                                 slab, slab_k, flag, status, s, gate);
    else
        launch_nlist_pass<true>(waves, kp, bv, n_blocks, n, x, x32, cell_start, rank_tab, offset, index, capacity,
                                slab, slab_k, flag, status, s, gate);
    return hipGetLastError();
}

hipError_t launch_nlist_compact(int32_t n, const int32_t* offset, int64_t capacity, const int32_t* slab,
                                int32_t slab_k, const int32_t* flag, int32_t* index, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_nlist_compact, dim3(ceil_div(ceil_div(n, kWave), kWavesPerBlock)), dim3(kBlock), 0, s, n,
                       offset, capacity, slab, slab_k, flag, index);
    return hipGetLastError();
}

}  // namespace dpd

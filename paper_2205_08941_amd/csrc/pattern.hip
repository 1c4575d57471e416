// Spatial-cutoff patterns: GPU cell-list neighbour search -> block CSR with
// sorted columns, transpose map and diagonal slots.
//
// The pattern is the locality structure of the paper's sparse matrices
// (Background and Current Status): an atom block (i, j) exists only when the
// minimum-image distance of atoms i and j is below the range of the operator.
#include "bsm_internal.h"

#include <algorithm>
#include <climits>
#include <cmath>

namespace bsm {
namespace {

constexpr int kMaxRow = 8192;   // longest row the LDS row sort handles

// Squared minimum-image distance, rounded exactly as written (no FMA), so the
// strict d^2 < r^2 decision is the one a plain CPU evaluation makes.
__device__ inline double min_image_d2(const double *__restrict__ pos, double bx, double by,
                                      double bz, int i, int j)
{
#pragma clang fp contract(off)
    const double box[3] = {bx, by, bz};
    double d2 = 0.0;
    for (int c = 0; c < 3; ++c) {
        double d = pos[3 * j + c] - pos[3 * i + c];
        double s = __builtin_rint(d / box[c]);
        d = d - s * box[c];
        d2 = d2 + d * d;
    }
    return d2;
}

struct Grid {
    int nc[3];
    int noff[3];   // neighbour offsets scanned per axis: 1, 2 or 3
    double box[3];
};

__device__ inline int cell_coord(double x, double box, int nc)
{
    double f = x / box;
    f -= floor(f);
    int c = (int)(f * nc);
    return c < 0 ? 0 : (c >= nc ? nc - 1 : c);
}

__global__ void k_cell_index(int n, const double *__restrict__ pos, Grid g, int *__restrict__ cell,
                             int *__restrict__ cellcount, int *__restrict__ nonfinite)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    if (!isfinite(pos[3 * i]) || !isfinite(pos[3 * i + 1]) || !isfinite(pos[3 * i + 2]))
        atomicOr(nonfinite, 1);
    int cx = cell_coord(pos[3 * i + 0], g.box[0], g.nc[0]);
    int cy = cell_coord(pos[3 * i + 1], g.box[1], g.nc[1]);
    int cz = cell_coord(pos[3 * i + 2], g.box[2], g.nc[2]);
    int c = (cx * g.nc[1] + cy) * g.nc[2] + cz;
    cell[i] = c;
    atomicAdd(&cellcount[c], 1);
}

// Exclusive scan of n ints into out[0..n] (out[n] = total) by one workgroup.
// Sets *overflow when the total does not fit in int32.
__global__ __launch_bounds__(1024) void k_scan(int n, const int *__restrict__ in, int *__restrict__ out,
                                               int *__restrict__ overflow)
{
    __shared__ long long part[1024];
    const int t = threadIdx.x, nt = blockDim.x;
    const int chunk = (n + nt - 1) / nt;
    const int lo = min(n, t * chunk), hi = min(n, lo + chunk);
    long long s = 0;
    for (int k = lo; k < hi; ++k) s += in[k];
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < nt; off <<= 1) {   // Hillis-Steele inclusive scan
        long long v = (t >= off) ? part[t - off] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    long long run = part[t] - s;
    for (int k = lo; k < hi; ++k) {
        out[k] = (int)run;
        run += in[k];
    }
    if (t == nt - 1) {
        out[n] = (int)part[t];
        *overflow = part[t] > (long long)INT_MAX ? 1 : 0;
    }
}

__global__ void k_cell_scatter(int n, const int *__restrict__ cell, const int *__restrict__ cellstart,
                               int *__restrict__ cellfill, int *__restrict__ cellatoms)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int c = cell[i];
    cellatoms[cellstart[c] + atomicAdd(&cellfill[c], 1)] = i;
}

constexpr int kNeighborThreads = 256;

// L lanes per atom: visit the neighbour cells, a lane per atom of a cell, and count
// (mode 0) or write (mode 1) the columns j with d^2 < r^2 (and j == i); the rows are sorted
// afterwards.  A thread per atom walked its cells alone, a chain of dependent loads and
// divisions: 78 and 96 us for 216 atoms at 8 A, 415 and 452 for 4096 at 10 A, against 6 and 6, 26 and 27.
template <int MODE, int L>
__global__ __launch_bounds__(kNeighborThreads) void k_neighbors(int n, const double *__restrict__ pos, Grid g,
                                                                  double r2, const int *__restrict__ cell,
                                                                  const int *__restrict__ cellstart,
                                                                  const int *__restrict__ cellatoms,
                                                                  int *__restrict__ rowcount,
                                                                  const int *__restrict__ rowptr,
                                                                  int *__restrict__ cols)
{
    const int i = blockIdx.x * (kNeighborThreads / L) + threadIdx.x / L, lane = threadIdx.x % L;
    if (i >= n) return;
    int c = cell[i];
    int cz = c % g.nc[2], cy = (c / g.nc[2]) % g.nc[1], cx = c / (g.nc[2] * g.nc[1]);
    int cnt = 0;
    int *row = (MODE == 1) ? cols + rowptr[i] : nullptr;
    // the atoms of the cells along z follow each other where the cells do: z cells as one or two runs
    const int first = (g.noff[2] == 3) ? cz - 1 : cz, last = first + g.noff[2];   // [first, last), wrapped
    for (int ox = 0; ox < g.noff[0]; ++ox) {
        int ax = (g.noff[0] == 3) ? cx + ox - 1 : cx + ox;
        ax = ((ax % g.nc[0]) + g.nc[0]) % g.nc[0];
        for (int oy = 0; oy < g.noff[1]; ++oy) {
            int ay = (g.noff[1] == 3) ? cy + oy - 1 : cy + oy;
            ay = ((ay % g.nc[1]) + g.nc[1]) % g.nc[1];
            const int base = (ax * g.nc[1] + ay) * g.nc[2];
            const int lo = max(first, 0), hi = min(last, g.nc[2]);
            const int q0 = cellstart[base + lo], n0 = cellstart[base + hi] - q0;
            // what wraps: below 0 the top cells, past the end the bottom ones (never both: noff <= nc)
            const int wl = first < 0 ? g.nc[2] + first : 0, wh = first < 0 ? g.nc[2] : last - hi;
            const int q1 = cellstart[base + wl], n1 = cellstart[base + wh] - q1;
            for (int x0 = 0; x0 < n0 + n1; x0 += L) {
                const int x = x0 + lane;
                bool near = false;
                int j = 0;
                if (x < n0 + n1) {
                    j = cellatoms[x < n0 ? q0 + x : q1 + (x - n0)];
                    near = j == i || min_image_d2(pos, g.box[0], g.box[1], g.box[2], i, j) < r2;
                }
                // the lanes of this atom: they run together
                const unsigned long long m = __ballot(near) >> (threadIdx.x % 64 / L * L) & (~0ull >> (64 - L));
                if (MODE == 1 && near) row[cnt + __popcll(m & ((1ull << lane) - 1ull))] = j;
                cnt += __popcll(m);
            }
        }
    }
    if (MODE == 0 && lane == 0) rowcount[i] = cnt;
}

// One workgroup per row: bitonic sort of the row's columns in LDS.
__global__ __launch_bounds__(256) void k_sort_rows(int n, const int *__restrict__ rowptr,
                                                   int *__restrict__ cols)
{
    __shared__ int v[kMaxRow];
    int i = blockIdx.x;
    if (i >= n) return;
    int lo = rowptr[i], len = rowptr[i + 1] - lo;
    int p2 = 1;
    while (p2 < len) p2 <<= 1;
    for (int t = threadIdx.x; t < p2; t += blockDim.x) v[t] = (t < len) ? cols[lo + t] : INT_MAX;
    __syncthreads();
    for (int k = 2; k <= p2; k <<= 1) {
        for (int jj = k >> 1; jj > 0; jj >>= 1) {
            for (int t = threadIdx.x; t < p2; t += blockDim.x) {
                int o = t ^ jj;
                if (o > t) {
                    bool up = (t & k) == 0;
                    int a = v[t], b = v[o];
                    if ((a > b) == up) {
                        v[t] = b;
                        v[o] = a;
                    }
                }
            }
            __syncthreads();
        }
    }
    for (int t = threadIdx.x; t < len; t += blockDim.x) cols[lo + t] = v[t];
}

__device__ inline int find_in_row(const int *__restrict__ rowptr, const int *__restrict__ cols, int i,
                                  int j)
{
    int lo = rowptr[i], hi = rowptr[i + 1], end = hi;
    while (lo < hi) {
        int mid = (lo + hi) >> 1;
        if (cols[mid] < j) lo = mid + 1;
        else hi = mid;
    }
    return (lo < end && cols[lo] == j) ? lo : -1;
}

__global__ void k_rows_of_slots(int n, const int *__restrict__ rowptr, int *__restrict__ rowidx)
{
    int i = blockIdx.x;
    if (i >= n) return;
    for (int s = rowptr[i] + threadIdx.x; s < rowptr[i + 1]; s += blockDim.x) rowidx[s] = i;
}

__global__ void k_tmap(int64_t nnz, const int *__restrict__ rowptr, const int *__restrict__ cols,
                       const int *__restrict__ rowidx, int *__restrict__ tmap, int *__restrict__ bad)
{
    int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nnz) return;
    int t = find_in_row(rowptr, cols, cols[s], rowidx[s]);
    tmap[s] = t;
    if (t < 0) *bad = 1;   // pinned host memory
}

__global__ void k_diag(int n, const int *__restrict__ rowptr, const int *__restrict__ cols,
                       int *__restrict__ diag)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) diag[i] = find_in_row(rowptr, cols, i, i);
}

// One workgroup: what the host needs to go on, in pinned memory: flags 0 .. 4, the longest
// row in place 2, and the number of slots in place 5.
__global__ __launch_bounds__(1024) void k_row_info(int n, const int *__restrict__ rowptr, const int *__restrict__ fl,
                                                   int *host)
{
    __shared__ int longest;
    if (threadIdx.x == 0) longest = 0;
    __syncthreads();
    int m = 0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) m = max(m, rowptr[i + 1] - rowptr[i]);
    for (int off = 32; off > 0; off >>= 1) m = max(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) atomicMax(&longest, m);
    __syncthreads();
    if (threadIdx.x < 6) host[threadIdx.x] = threadIdx.x == 2 ? longest : threadIdx.x == 5 ? rowptr[n] : fl[threadIdx.x];
}

inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

bsm_pattern_s *make_pattern(Context *ctx, int natoms, int b, const double *pos_dev, const double box[3],
                            double cutoff)
{
    BSM_REQUIRE(natoms > 0, BSM_EINVAL, "natoms must be positive");
    BSM_REQUIRE(b >= 1 && b <= 16, BSM_EINVAL, "b must be in 1..16");
    BSM_REQUIRE(cutoff > 0 && std::isfinite(cutoff), BSM_EINVAL, "cutoff must be positive");
    BSM_REQUIRE(pos_dev != nullptr, BSM_EINVAL, "positions are NULL");
    for (int d = 0; d < 3; ++d)
        BSM_REQUIRE(box[d] > 0 && std::isfinite(box[d]), BSM_EINVAL, "box must be positive");

    hipStream_t st = ctx->stream;
    std::unique_ptr<bsm_pattern_s> p(new bsm_pattern_s());
    p->ctx = ctx;
    p->id = ctx->next_pattern_id++;
    p->natoms = natoms;
    p->b = b;
    p->cutoff = cutoff;
    for (int d = 0; d < 3; ++d) p->box[d] = box[d];
    p->pos = DevBuf(ctx, sizeof(double) * 3 * (size_t)natoms);
    BSM_HIP_TRY(hipMemcpyAsync(p->pos.ptr, pos_dev, sizeof(double) * 3 * (size_t)natoms,
                               hipMemcpyDeviceToDevice, st));

    Grid g;
    int64_t ncells = 1;
    for (int d = 0; d < 3; ++d) {
        double q = std::floor(box[d] / cutoff);
        int nc = (int)std::max(1.0, std::min(q, 256.0));
        g.nc[d] = nc;
        g.noff[d] = nc >= 3 ? 3 : nc;
        g.box[d] = box[d];
        ncells *= nc;
    }

    const size_t ra = Cut::room(sizeof(int) * natoms), rc = Cut::room(sizeof(int) * ncells);
    DevBuf work(ctx, 256 + 2 * rc + Cut::room(sizeof(int) * (ncells + 1)) + 3 * ra);
    Cut cut{work.as<char>()};
    int *fl = cut.take<int>(8), *cellcount = cut.take<int>(ncells), *cellfill = cut.take<int>(ncells);
    BSM_HIP_TRY(hipMemsetAsync(work.ptr, 0, cut.used, st));   // flags and counts
    int *cellstart = cut.take<int>(ncells + 1), *cell = cut.take<int>(natoms), *cellatoms = cut.take<int>(natoms),
        *rowcount = cut.take<int>(natoms);

    k_cell_index<<<blocks_for(natoms, 256), 256, 0, st>>>(natoms, p->pos.as<double>(), g, cell,
                                                            cellcount, fl + 4);
    k_scan<<<1, 1024, 0, st>>>((int)ncells, cellcount, cellstart, fl + 0);
    k_cell_scatter<<<blocks_for(natoms, 256), 256, 0, st>>>(natoms, cell, cellstart,
                                                              cellfill, cellatoms);
    double r2 = cutoff * cutoff;
    // Lanes of an atom: a wavefront of 64 mostly idles where a run of cells along z holds few
    // atoms, and many atoms fill the chip with 16 lanes each.  The whole pattern, 16 lanes and 64:
    // 4096 atoms, 6 A (36 atoms a run) 150 and 152 us, 8 A (98) 213 and 181; 32768 atoms, 4 A (11)
    // 309 and 409, 10 A (192) 1016 and 1046; 327680 atoms, 4 A (10) 2355 and 3401, a thread per atom 2411.
    const double run = (double)natoms / (double)ncells * g.noff[2];
    const bool narrow = run <= 40.0 || natoms >= 16384;
    auto neighbors = [&](auto MODE, int *count, const int *rowptr, int *cols) {
        auto go = [&](auto kern, int lanes) {
            kern<<<blocks_for(natoms, kNeighborThreads / lanes), kNeighborThreads, 0, st>>>(
                natoms, p->pos.as<double>(), g, r2, cell, cellstart, cellatoms, count, rowptr, cols);
        };
        constexpr int mode = decltype(MODE)::value;
        narrow ? go(k_neighbors<mode, 16>, 16) : go(k_neighbors<mode, 64>, 64);
    };
    neighbors(std::integral_constant<int, 0>{}, rowcount, nullptr, nullptr);
    p->rowptr = DevBuf(ctx, sizeof(int) * (natoms + 1));
    k_scan<<<1, 1024, 0, st>>>(natoms, rowcount, p->rowptr.as<int>(), fl + 1);
    int *hostv = reinterpret_cast<int *>(ctx->host_scalars + kHostCounts);
    k_row_info<<<1, 1024, 0, st>>>(natoms, p->rowptr.as<int>(), fl, hostv);
    BSM_HIP_TRY(hipGetLastError());
    BSM_HIP_TRY(hipStreamSynchronize(st));
    const int total = hostv[5];
    BSM_REQUIRE(hostv[4] == 0, BSM_EINVAL, "positions are not finite");
    BSM_REQUIRE(hostv[1] == 0, BSM_EINVAL, "pattern has more than 2^31-1 blocks");
    BSM_REQUIRE(hostv[2] <= kMaxRow, BSM_EINVAL, "a pattern row is longer than 8192 blocks");
    p->nnzb = total;
    p->max_row = hostv[2];

    p->cols = DevBuf(ctx, sizeof(int) * (size_t)total);
    neighbors(std::integral_constant<int, 1>{}, nullptr, p->rowptr.as<int>(), p->cols.as<int>());
    k_sort_rows<<<natoms, 256, 0, st>>>(natoms, p->rowptr.as<int>(), p->cols.as<int>());

    p->rowidx = DevBuf(ctx, sizeof(int) * (size_t)total);
    k_rows_of_slots<<<natoms, 64, 0, st>>>(natoms, p->rowptr.as<int>(), p->rowidx.as<int>());
    p->tmap = DevBuf(ctx, sizeof(int) * (size_t)total);
    p->diag = DevBuf(ctx, sizeof(int) * natoms);
    hostv[0] = 0;
    k_tmap<<<blocks_for(total, 256), 256, 0, st>>>(total, p->rowptr.as<int>(), p->cols.as<int>(),
                                                   p->rowidx.as<int>(), p->tmap.as<int>(), hostv);
    k_diag<<<blocks_for(natoms, 256), 256, 0, st>>>(natoms, p->rowptr.as<int>(), p->cols.as<int>(),
                                                    p->diag.as<int>());
    BSM_HIP_TRY(hipGetLastError());
    BSM_HIP_TRY(hipStreamSynchronize(st));
    BSM_REQUIRE(hostv[0] == 0, BSM_EINVAL, "pattern is not symmetric (non-finite positions?)");
    return p.release();
}

bsm_pattern_s *derived_pattern(const bsm_pattern_s *p, double cutoff)
{
    return make_pattern(p->ctx, p->natoms, p->b, p->pos.as<double>(), p->box, cutoff);
}

const bsm_pattern_s *derived_pattern_cached(const bsm_pattern_s *p, double cutoff)
{
    Context *ctx = p->ctx;
    auto key = std::make_pair(p->id, cutoff);
    auto it = ctx->derived.find(key);
    if (it != ctx->derived.end()) return it->second;
    bsm_pattern_s *d = derived_pattern(p, cutoff);
    ctx->derived[key] = d;
    return d;
}

void destroy_pattern(bsm_pattern_s *p)
{
    if (!p) return;
    Context *ctx = p->ctx;
    // patterns derived from this one go first
    std::vector<bsm_pattern_s *> kids;
    for (auto it = ctx->derived.begin(); it != ctx->derived.end();) {
        if (it->first.first == p->id) {
            kids.push_back(it->second);
            it = ctx->derived.erase(it);
        } else {
            ++it;
        }
    }
    for (bsm_pattern_s *k : kids) destroy_pattern(k);
    ctx->forget_pattern(p->id);
    delete p;
}

}  // namespace bsm

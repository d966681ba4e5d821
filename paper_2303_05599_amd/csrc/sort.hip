// sort.hip -- periodic reordering of the particle records by lattice cell.
//
// The push gathers the fields around each particle's nearest grid point, and
// the fused step (fused.hip) pushes the particles of a tile in the workgroup
// that updates the tile.  Particles are ordered by tiles of tx x ty cells
// (tile-major, then row-major inside the tile): 32 x 16 for the gather push,
// whose wavefronts and the workgroups that run together on one XCD then read
// a compact patch of the lattice in whole cache lines, and the fused kernel's
// own tile shape for the fused step, which also receives the range of records
// of every tile.  The key of a moving particle is its nearest grid point at
// the step the order is made for (from its position), of a static one its
// cell.  The order is that of a stable sort of the keys (a counting sort,
// below); the records are copied aside and moved from there to their places so
// that buffer addresses (captured in HIP graphs) never change.  pid tracks
// each record's original index for state exchange.
//
// The sort is stable and the same on every run.  It is launch-bound up to some
// 1e5 records: two launches for few records (their number squared, until five are
// cheaper: a step at 8192 records took 17.2 us with two, 17.0 with five), five
// otherwise.  Kernel time of one reordering against seven launches (a library
// scan, a pass that sorts the run of every key, a permutation into the scratch
// copy and a copy back): 3000 records at 96^2 33 -> 12 us, 16329 at 216^2 (FP64) 35
// -> 25, 1e6 at 512^2 (FP32) 252 -> 174, where moving 84 MB of records twice sets
// the pace.
#include "internal.h"

namespace cpic {

__host__ __device__ inline unsigned sort_key_bound(int N, int tx, int ty)
{
    return (unsigned)fused_tiles(N, tx, ty) * (unsigned)(tx * ty);
}

// blocks of 256, consecutive ones on one XCD
__device__ __forceinline__ int band_block(int nblocks)
{
    const int per = (nblocks + 7) / 8;
    return ((int)blockIdx.x & 7) * per + ((int)blockIdx.x >> 3);
}
static dim3 banded(int nblocks) { return dim3(8 * ((nblocks + 7) / 8)); }

// The key of every record, and the record copied to the scratch buffers it is
// moved from.  COUNT: the number of records of each key, and the record's place
// among those of its key, in the order the increments happened in.
template <typename T, bool COUNT>
__global__ __launch_bounds__(256) void cell_keys_kernel(const T* __restrict__ r, const int* __restrict__ cell,
                                                        const int* __restrict__ pid, int np, int N, int tx, int ty,
                                                        int from_position, unsigned* keys, int* count, int* slot,
                                                        T* r2, int* cell2, int* pid2)
{
    const int p = blockIdx.x * 256 + threadIdx.x;
    if (p >= np) return;
    T v[kPartReals];
#pragma unroll
    for (int c = 0; c < kPartReals; c++) v[c] = r[(size_t)c * np + p];
    const int ox = cell[p], oy = cell[np + p], id = pid[p];
    int cx = ox, cy = oy;
    if (from_position) {
        // the nearest grid point as the push computes it
        const int nx = (int)floor(v[PX_] + T(0.5)), ny = (int)floor(v[PY_] + T(0.5));
        cx = nx >= N ? nx - N : nx;
        cy = ny >= N ? ny - N : ny;
    }
    // a non-finite position (a diverged run, which the watchdog reports) still
    // gets a key inside the lattice's range
    cx = min(max(cx, 0), N - 1);
    cy = min(max(cy, 0), N - 1);
    const int ntx = (N + tx - 1) / tx;
    const int tile = (cy / ty) * ntx + cx / tx;
    const unsigned key = (unsigned)(tile * tx * ty + (cy % ty) * tx + cx % tx);
    keys[p] = key;
    if constexpr (COUNT) {
        slot[p] = atomicAdd(&count[key], 1);
    }
#pragma unroll
    for (int c = 0; c < kPartReals; c++) r2[(size_t)c * np + p] = v[c];
    cell2[p] = ox;
    cell2[np + p] = oy;
    pid2[p] = id;
}

// Few records: the place of each is the number of records before it, counted
// over all keys by one wavefront, which then moves the record.
constexpr int kRankMax = 4096;
template <typename T>
__global__ __launch_bounds__(256) void rank_move_kernel(const unsigned* __restrict__ keys, int np,
                                                        const T* __restrict__ r2, const int* __restrict__ cell2,
                                                        const int* __restrict__ pid2, unsigned* keys2, T* r, int* cell,
                                                        int* pid)
{
    const int i = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 256 + threadIdx.x) >> 6);
    const int s = (int)threadIdx.x & 63;
    if (i >= np) return;
    const unsigned ki = keys[i];
    int before = 0;
    // j < i: equal keys count as well
    auto add = [&](unsigned k, int j) { before += k < ki + (j < i ? 1u : 0u) ? 1 : 0; };
    const int quads = np / 4;
#pragma unroll 4
    for (int q = s; q < quads; q += 64) {
        const uint4 k = reinterpret_cast<const uint4*>(keys)[q];
        add(k.x, 4 * q);
        add(k.y, 4 * q + 1);
        add(k.z, 4 * q + 2);
        add(k.w, 4 * q + 3);
    }
    if (4 * quads + s < np) add(keys[4 * quads + s], 4 * quads + s);
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) before += __shfl_xor(before, m);
    if (s == 0) keys2[before] = ki;
    // one lane per column: the reals, the cell, the input index
    if (s < kPartReals) r[(size_t)s * np + before] = r2[(size_t)s * np + i];
    else if (s < kPartReals + 2) cell[(size_t)(s - kPartReals) * np + before] = cell2[(size_t)(s - kPartReals) * np + i];
    else if (s == kPartReals + 2) pid[before] = pid2[i];
}

// tile_start[t] = first record of tile t (or of the next non-empty tile),
// tile_start[ntiles] = np, from the sorted keys; every entry is written once
__global__ void tile_start_kernel(const unsigned* __restrict__ sorted, int np, unsigned per_tile, int ntiles,
                                  int* tile_start)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > np) return;
    const int ti = i < np ? (int)min(sorted[i] / per_tile, (unsigned)ntiles) : ntiles;
    const int tp = i > 0 ? (int)min(sorted[i - 1] / per_tile, (unsigned)ntiles) : -1;
    for (int t = tp + 1; t <= ti; t++) tile_start[t] = i;
}

// Many records: a counting sort of the keys (dense integers below
// key_capacity(N)).  The counts are added up per chunk of keys first (by a kernel of
// its own: counted beside the keys, a few hundred contended addresses took 800 us
// for 1e6 records).
constexpr int kChunk = 512;
__global__ __launch_bounds__(256) void chunk_counts_kernel(const int* __restrict__ count, int nkeys, int* chunk)
{
    __shared__ int part[4];
    const int t = (int)threadIdx.x, k = (int)blockIdx.x * kChunk + 2 * t;
    int n = (k < nkeys ? count[k] : 0) + (k + 1 < nkeys ? count[k + 1] : 0);
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) n += __shfl_xor(n, m);
    if ((t & 63) == 0) part[t >> 6] = n;
    __syncthreads();
    if (t == 0) chunk[blockIdx.x] = part[0] + part[1] + part[2] + part[3];
}
// Exclusive sums of the counts, one workgroup per chunk of keys, which adds up the
// chunks before its own; it clears the counts it read, so that they are zero
// between reorderings (and from allocation on), and writes the range of records of
// every tile.
__global__ __launch_bounds__(256) void chunk_sums_kernel(int* count, const int* __restrict__ chunk, int nkeys, int np,
                                                         int per_tile, int* offs, int* tile_start)
{
    __shared__ int part[4], run[4];
    const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6, c = (int)blockIdx.x;
    int base = 0;
    for (int j = t; j < c; j += 256) base += chunk[j];
    const int k = c * kChunk + 2 * t;
    const int n0 = k < nkeys ? count[k] : 0, n1 = k + 1 < nkeys ? count[k + 1] : 0;
    if (k < nkeys) count[k] = 0;
    if (k + 1 < nkeys) count[k + 1] = 0;
    int incl = n0 + n1;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        base += __shfl_xor(base, m);
        const int v = __shfl_up(incl, m);
        incl += lane >= m ? v : 0;
    }
    if (lane == 63) run[wave] = incl;
    if (lane == 0) part[wave] = base;
    __syncthreads();
    int at = part[0] + part[1] + part[2] + part[3] + incl - n0 - n1;
#pragma unroll
    for (int w = 0; w < 3; w++) at += w < wave ? run[w] : 0;
#pragma unroll
    for (int h = 0; h < 2; h++) {
        if (k + h < nkeys) {
            offs[k + h] = at;
            if (tile_start && (k + h) % per_tile == 0) tile_start[(k + h) / per_tile] = at;
        }
        if (k + h == nkeys - 1) {
            offs[nkeys] = np;
            if (tile_start) tile_start[nkeys / per_tile] = np;
        }
        at += n0;
    }
}
// the records of every key side by side, in the order of their increments
__global__ __launch_bounds__(256) void group_kernel(const unsigned* __restrict__ keys, const int* __restrict__ slot,
                                                    const int* __restrict__ offs, int np, int nblocks, int* perm)
{
    const int blk = band_block(nblocks), p = blk * 256 + (int)threadIdx.x;
    if (blk >= nblocks || p >= np) return;
    perm[offs[keys[p]] + slot[p]] = p;
}
// The place of a record among those of its key is the number of them with a
// smaller index (a few records per cell; many piled on one cell cost their number
// squared, spread over as many threads).  Its neighbours in the last order are
// its neighbours in the new one but for a few rows of a tile: consecutive blocks
// on one XCD find them in its L2.
template <typename T>
__global__ __launch_bounds__(256) void move_kernel(const unsigned* __restrict__ keys, const int* __restrict__ offs,
                                                   const int* __restrict__ perm, int np, int nblocks,
                                                   const T* __restrict__ r2, const int* __restrict__ cell2,
                                                   const int* __restrict__ pid2, unsigned* keys2, T* r, int* cell,
                                                   int* pid)
{
    const int blk = band_block(nblocks), i = blk * 256 + (int)threadIdx.x;
    if (blk >= nblocks || i >= np) return;
    const int src = perm[i];
    const unsigned k = keys[src];
    const int begin = offs[k], end = offs[k + 1];
    int dst = begin;
    for (int j = begin; j < end; j++) dst += perm[j] < src ? 1 : 0;
    keys2[i] = k;
#pragma unroll
    for (int c = 0; c < kPartReals; c++) r[(size_t)c * np + dst] = r2[(size_t)c * np + src];
    cell[dst] = cell2[src];
    cell[np + dst] = cell2[np + src];
    pid[dst] = pid2[src];
}

__global__ void iota_kernel(int* p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = i;
}
hipError_t launch_iota(int* p, int n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(iota_kernel, dim3((n + 255) / 256), dim3(256), 0, st, p, n);
    return hipGetLastError();
}

int key_capacity(int N)
{
    // the largest key bound of any tile shape (tiles of at most 64 x 64 cells)
    return (N + 64) * (N + 64);
}

int key_chunks(int N) { return (key_capacity(N) + kChunk - 1) / kChunk; }

hipError_t launch_tile_start(const unsigned* sorted_keys, int np, int N, int tx, int ty, int* tile_start,
                             hipStream_t st)
{
    if (np <= 0 || !fused_shape(tx, ty)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(tile_start_kernel, dim3((np + 256) / 256), dim3(256), 0, st, sorted_keys, np,
                       (unsigned)(tx * ty), fused_tiles(N, tx, ty), tile_start);
    return hipGetLastError();
}

template <typename T>
hipError_t sort_particles(const SortBufs& b, T* r, int* cell, int* pid, int np, int N, int tx, int ty,
                          bool from_position, int* tile_start, hipStream_t st)
{
    if (np <= 0 || tx <= 0 || ty <= 0) return np <= 0 ? hipSuccess : hipErrorInvalidValue;
    const unsigned nkeys = sort_key_bound(N, tx, ty);
    if (nkeys > (unsigned)b.key_cap) return hipErrorInvalidValue;
    const int blocks = (np + 255) / 256, pos = from_position ? 1 : 0;
    T* const r2 = static_cast<T*>(b.r2);
    if (np <= kRankMax) {
        hipLaunchKernelGGL((cell_keys_kernel<T, false>), dim3(blocks), dim3(256), 0, st, r, cell, pid, np, N, tx, ty,
                           pos, b.keys, nullptr, nullptr, r2, b.cell2, b.pid2);
        hipLaunchKernelGGL(rank_move_kernel<T>, dim3((np + 3) / 4), dim3(256), 0, st, b.keys, np, r2, b.cell2,
                           b.pid2, b.keys2, r, cell, pid);
        if (tile_start) return launch_tile_start(b.keys2, np, N, tx, ty, tile_start, st);
        return hipGetLastError();
    }
    const int nchunks = (int)((nkeys + kChunk - 1) / kChunk);
    int* const slot = b.perm + np;
    int* const chunk = b.count + b.key_cap;
    hipLaunchKernelGGL((cell_keys_kernel<T, true>), dim3(blocks), dim3(256), 0, st, r, cell, pid, np, N, tx, ty, pos,
                       b.keys, b.count, slot, r2, b.cell2, b.pid2);
    hipLaunchKernelGGL(chunk_counts_kernel, dim3(nchunks), dim3(256), 0, st, b.count, (int)nkeys, chunk);
    hipLaunchKernelGGL(chunk_sums_kernel, dim3(nchunks), dim3(256), 0, st, b.count, chunk, (int)nkeys, np, tx * ty,
                       b.offs, tile_start);
    hipLaunchKernelGGL(group_kernel, banded(blocks), dim3(256), 0, st, b.keys, slot, b.offs, np, blocks, b.perm);
    hipLaunchKernelGGL(move_kernel<T>, banded(blocks), dim3(256), 0, st, b.keys, b.offs, b.perm, np, blocks, r2,
                       b.cell2, b.pid2, b.keys2, r, cell, pid);
    return hipGetLastError();  // launch errors surface at the stream's next synchronisation, as for every kernel
}

template hipError_t sort_particles<double>(const SortBufs&, double*, int*, int*, int, int, int, int, bool, int*,
                                           hipStream_t);
template hipError_t sort_particles<float>(const SortBufs&, float*, int*, int*, int, int, int, int, bool, int*,
                                          hipStream_t);

}  // namespace cpic

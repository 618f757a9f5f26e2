// Batched activation-checkpoint dynamic program on gfx950: kernels and C ABI.
//
// Computes C_BP(s, t, m) of the paper's Theorem (Section "Activation Checkpoint
// Solver / Modeling") for B chains at once.  See include/ckpt_dp.h for the
// conventions (candidate numbering, saturation at 2^30, table layout).
#include <hip/hip_runtime.h>

#include <array>
#include <atomic>
#include <utility>
#include <cstdint>
#include <cstring>
#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "ckpt_rules.h"
#include "ckpt_dp.h"

namespace {

constexpr uint32_t kInf = 1u << 30;
constexpr int kT = 8;  // stage-block size of the fill
constexpr int kCH = 2;  // 64-column chunks of m per gemm work-group
constexpr int kRowWG = 256;  // threads (columns of m) per work-group of the row kernels
std::atomic<int> g_last_hip_error{0};

inline bool hip_ok(hipError_t e) {
    if (e != hipSuccess) {
        g_last_hip_error.store(static_cast<int>(e));
        return false;
    }
    return true;
}

// ---------------------------------------------------------------------------
// How the table is filled
//
// Stages are 0-based inside this file: cell (i, j), 0 <= i <= j < L, is the paper's
// (s, t) = (i + 1, j + 1).  A checkpoint split q in i+1..j is the paper's s' = q + 1:
// left operand cell (i, q-1) at the same m, right operand cell (q, j) at m - omega_a^q,
// plus the forward sweep P[q] - P[i] (C_ck of the Theorem).  Its candidate number is q + 1.
//
// Stages are grouped in blocks of T.  Tile (I, J) holds the cells with i in block I and
// j in block J.  Tiles are processed by block diagonal D = J - I; within one D every
// tile is independent.  The splits of a cell of tile (I, J), D >= 2, fall in three groups:
//   middle   q in [(I+1)T, JT]: both operands lie in tiles of a smaller D.  This is a
//            min-plus product of a register tile of cells per lane (gemm_kernel), where each
//            loaded operand row is reused by all cells of a row or column of the tile.
//   near-i   q in block I: the right operand (q, j) is a lower row of the SAME tile, read
//            at a shifted m, so the rows of a tile are finished bottom-up.
//   near-j   q in block J: the left operand (i, q-1) is an earlier cell of the same row at
//            the same m, kept in registers.
// A row is finished by its near-i splits, the partial minimum of gemm_kernel, its near-j splits, then C_all and the
// two gates.  Launch order per D: gemm (D >= 2), which also finishes row T-1, then tile_rows_kernel, one launch for
// rows T-2 .. 0 (T-1 .. 0 for D < 2) of every tile.  row_kernel, one launch per row, is the alternative schedule.
// Batches that leave the chip half empty take all tiles in one launch (flow_kernel), short chains are one launch altogether
// (chain_kernel); ckpt_rules.h says which.
//
// Reads at m - shift are not bounds-checked against m < shift: a lane whose m is below
// a shift of one of its splits is below m_null (m_all for C_all) of that cell, because
// both thresholds contain every shift of the cell, so the gate discards whatever it
// read.  Shifts are clamped to one row pitch, which keeps such reads inside the table.
// ---------------------------------------------------------------------------

// Workspace layout, all per chain b:
//   P     [B][L+1] int32   P[i] = sum of u_f of stages 1..i
//   fb    [B][L]   int32   min(2^30, u_f + u_b) of stage i+1
//   wsh   [B][L]   int32   shift of split q: omega_a^q clamped to [0, pitch]
//   wabs  [B][L]   int32   shift of C_all at row i: omega_abar^{i+1} clamped to [0, pitch]
//   mall  [B][L][L] int32  m_all^{s,t}  at [i*L + j]
//   mnull [B][L][L] int32  m_null^{s,t}
//   flags [B]      int32   input precondition flags
//   need  [B][L][L] int32  feasibility frontier: smallest m at which cell (i, j) can be finite
//   prog  [B][tiles][chunks + 1] int32  rows of tile (I, J) finished by tile_rows_kernel for the chunk
//                          of 64 columns; tiles = nblk (nblk + 1) / 2, chunks = pitch / 64; last word: bands of
//                          the tile that work-groups have taken.  flow_kernel: 1 where the tile is finished; last
//                          words: of the first tile, tickets of the chain; of the last one, the chain's largest shift
//   fault [1]      int32   set when a bounded wait inside tile_rows_kernel or flow_kernel expired
//   samp  [B][4 nblk (nblk + 1)][pitch / kG][8] int32  every kG-th column of the finished cells, eight cells of a
//                          row side by side (see gemm_kernel); left out where they are not used or do not fit
// prog and fault are cleared by precompute_kernel at the start of every solve.  chain_kernel uses flags and fault only.
struct Workspace {
    int32_t* P;
    int32_t* fb;
    int32_t* wsh;
    int32_t* wabs;
    int32_t* mall;
    int32_t* mnull;
    int32_t* flags;
    int32_t* need;
    int32_t* prog;
    int32_t* fault;
    int32_t* samp;  // null: no samples are kept
};

using ckpt_rules::kG;  // columns between samples
constexpr double kKeyBase = 0x1p44;

constexpr int kBand = kRowWG;  // columns of m per work-group of the row kernels

inline size_t align64(size_t n) { return (n + 63) & ~size_t(63); }
__host__ __device__ inline int blocks_of(int L) { return (L + kT - 1) / kT; }
__host__ __device__ inline size_t tiles_of(int L) { return size_t(blocks_of(L)) * (blocks_of(L) + 1) / 2; }
__host__ __device__ inline int bands_of(int pitch) { return (pitch + kBand - 1) / kBand; }
// index of tile (I, J), I <= J, in the row-major packed block triangle
__host__ __device__ inline int tile_index(int nblk, int I, int J) { return I * nblk - (I * (I - 1)) / 2 + (J - I); }

// Samples of one chain: [samp_rows][pitch / kG][8], cell (i, j) in row 4 J (J + 1) + i of column block J = j / 8.
__host__ __device__ inline int samp_rows(int L) { return 4 * blocks_of(L) * (blocks_of(L) + 1); }
__host__ __device__ inline size_t samp_ints(int L, int pitch) {
    return blocks_of(L) < 3 ? 0 : size_t(pitch / kG) * samp_rows(L) * kT;
}

// Whether the block product bounds its splits by samples (else it evaluates every feasible one).  The bounds are two
// more chains of dependent reads a launch, which pay where the launches have enough splits, about
// B pitch nblk^2 / 8 on average, and where kG columns are a small part of the budget: the narrower the table,
// the more a cost varies over a sub-chunk and the less the bounds drop.  The line was drawn through 295 shapes, each
// timed with and without.  It is within 0.3 % of the better one on average (2e5 .. 6.4e6 by that measure, five mixes of
// stages), and at worst 11 % (43 x 192 stages of nearly one size in 124 slots: the bounds drop little).  Both sides, without and with:
//   one chunk of columns: 49 x 254 stages, 60 slots (3.2e6) 2857 us and 3232; 300 x 254 (2e7) 15.0 ms and 16.4
//   three blocks: 289 x 24 stages, 565 slots (1.5e6) 196 us and 205; 1068 x 24, 4096 slots (4e7) 4477 and 4404
//   four blocks: 137 x 32 stages, 318 slots (7.0e5) 157 and 160; 23 x 32, 4088 slots (1.5e6) 256 and 250
//   narrow: 6 x 254 stages, 124 slots (7.9e5) 1633 and 1738; 14 x 192, 188 slots (1.5e6) 1318 and 1253; 10 x 96, 303
//   slots (4.6e5) 424 and 443; 20 x 128, 316 slots (1.6e6) 900 and 798
//   else: 5 x 53 stages, 777 slots (2.0e5) 239 and 249; 1 x 254, 500 slots (5.2e5) 1611 and 1739; 4 x 77, 999 slots (4.1e5)
//   382 and 391; 1 x 128, 2048 slots (5.4e5) 633 and 618; 3 x 80, 2273 slots (6.9e5) 402 and 388; 1 x 128, 1719 slots
//   (4.4e5) 610 and 582; 6 x 96, 1147 slots (10e5) 529 and 500
// A batch with bounds has them with more chains, stages or columns too, so a workspace serves every smaller batch.
inline bool uses_bounds(int L, int pitch, int B) {
    const int nblk = blocks_of(L);
    if (nblk < 3 || pitch <= 64) return false;
    const double line = nblk == 3 ? 2e7 : nblk == 4 ? 1.4e6 : std::max(4e5, std::min(1.4e6, 4.5e8 / pitch));
    return double(B) * pitch * nblk * nblk >= line;
}

__host__ __device__ inline int prog_words(int pitch) { return pitch / 64 + 1; }
inline size_t ws_ints(int L, int pitch, int B) {
    return align64(size_t(B) * (L + 1)) + 3 * align64(size_t(B) * L) + 3 * align64(size_t(B) * L * L) +
           align64(size_t(B)) + align64(size_t(B) * tiles_of(L) * prog_words(pitch)) + 64;
}
// The measure by which ckpt_solve_batched_noalloc accepts a call.  It is the size of a layout with two more words a
// stage, four a block and none for the tickets of the tiles, kept so that the calls which are accepted stay
// the same.  ws_ints exceeds it by less than tiles - 2 L words a chain, which is positive for 32 blocks only, at
// most 30, and no more than 22 such chains are accepted: kScratchSlack holds that.
inline size_t limit_ints(int L, int pitch, int B) {
    return ws_ints(L, pitch, B) - align64(size_t(B) * tiles_of(L) * prog_words(pitch)) +
           align64(size_t(B) * tiles_of(L) * (pitch / 64)) + 2 * align64(size_t(B) * L) + align64(size_t(blocks_of(L)) * 4);
}
constexpr size_t kScratchSlack = 4096;
static_assert(CKPT_MAX_L <= 256 && kScratchSlack >= 22 * 30 * sizeof(int32_t), "see limit_ints");

inline bool samples_of(int L, int pitch, int B) { return uses_bounds(L, pitch, B) && samp_ints(L, pitch); }

inline Workspace carve(void* base, int L, int pitch, int B, bool samples) {
    int32_t* p = static_cast<int32_t*>(base);
    Workspace w;
    w.P = p;      p += align64(size_t(B) * (L + 1));
    w.fb = p;     p += align64(size_t(B) * L);
    w.wsh = p;    p += align64(size_t(B) * L);
    w.wabs = p;   p += align64(size_t(B) * L);
    w.mall = p;   p += align64(size_t(B) * L * L);
    w.mnull = p;  p += align64(size_t(B) * L * L);
    w.flags = p;  p += align64(size_t(B));
    w.need = p;   p += align64(size_t(B) * L * L);
    w.prog = p;   p += align64(size_t(B) * tiles_of(L) * prog_words(pitch));
    w.fault = p;  p += 64;
    w.samp = samples && samples_of(L, pitch, B) ? p : nullptr;
    return w;
}

struct Ctx {
    int L, M, pitch, rows;
    int b0;  // first chain of this launch; blockIdx.z counts from it
    int spin_limit;  // polls before a wait between work-groups gives up; < 0: every such wait gives up at once
    Workspace ws;
    int32_t* cost;
    uint8_t* arg;
    // measurement only (ckpt_solve_profiled), else null: kWorkSets sets of four counters, [0] bytes
    // of table loads the gemm's waves asked for, [1] bytes they stored, [2], [3] the same for the
    // row kernel; a wave adds to the set its position selects, the host sums the sets
    unsigned long long* work;
    bool passing;  // rows of the block product are stored as passing through the caches (see rows_pass)
};
constexpr int kWorkSets = 256;

// One lane per wave adds the wave's byte counts (per lane 4 bytes a load, 5 a stored cell).  gemm_kernel and tile_rows_kernel count
// in instantiations of their own, at no cost otherwise; flow_kernel (a work-group once) and chain_kernel (a row) ask at run time.
template <bool CNT>
__device__ __forceinline__ void count_work(unsigned long long* work, int slot, unsigned loads, unsigned cells) {
    if constexpr (!CNT) return;
    if (work && (threadIdx.x & 63) == 0) {
        const unsigned set = (blockIdx.x * 7u + blockIdx.y * 13u + blockIdx.z * 29u + (threadIdx.x >> 6)) % kWorkSets;
        atomicAdd(work + set * 4 + slot, 256ull * loads);
        atomicAdd(work + set * 4 + slot + 1, 320ull * cells);
    }
}

__host__ __device__ inline int tri_row(int L, int i, int j) {  // 0-based i <= j
    return i * L - (i * (i - 1)) / 2 + (j - i);
}

constexpr uint32_t kNoRead = 0xfffffff0u;  // buffer offset beyond any table: the load returns 0, no access

// Inclusive scan over the 64 lanes of a wave; 0 is the identity of op.
template <class Op>
__device__ __forceinline__ int wave_scan(int v, Op op) {
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false));  // one, two, four, eight lanes before, in a row of 16
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false));
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false));
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false));
    v = op(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false));     // the end of rows 0 and 2 to rows 1 and 3
    return op(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false));  // the end of row 1 to rows 2 and 3
}

// Input checks, prefix sums, shifts and both threshold tables (last display of the Theorem), and for flow_kernel the marks
// of the first diagonal's tiles.  A chain has `parts` work-groups with `rows` rows of the tables each, one for what there
// is once per chain, and those that mark.  Rows have a thread per column t: the maximum over the stages
// between s and t is a scan for the lowest row and grows by one stage from row to row, and the rows are written in whole
// lines.  What bounds it: a launch, one round trip to memory and some hundred instructions of a lone wave; with
// thousands of chains the start of work-groups, so these have the waves that the stages fill (marks need all four).
// 8 chains of 192 stages: 6.6 us, 18.0 with sixteen rows and a loop over the stages above them, by work-groups of which
// one had the chain's part too; 10 chains of 50: 4.2 and 8.6, 1 of 8: 2.7 and 4.0, 20000 of 8: 23 and 40.
constexpr int kPreThreads = 256, kMarkCols = 512;
constexpr uint32_t kMark = 0x80000000u;  // a cell that waits for its row
static_assert(CKPT_MAX_L < kPreThreads, "a thread per stage");

__global__ void __launch_bounds__(kPreThreads) precompute_kernel(ckpt_chains_t ch, int L, int pitch, Workspace ws, int rows,
                                                                  int parts, int32_t* cost) {
    const int b = blockIdx.x, part = blockIdx.y;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool flow = int(gridDim.y) > parts + 1;  // for flow_kernel
    if (part > parts) {  // marks kMarkCols columns of rows 1 .. 7 of a tile of the first diagonal
        const int segs = (pitch + kMarkCols - 1) / kMarkCols, seg = part - parts - 1;
        const int I = seg / segs, m = seg % segs * kMarkCols + 4 * (tid & 127);
        int4* at = reinterpret_cast<int4*>(cost + size_t(b) * (size_t(L) * (L + 1) / 2) * pitch + m);
        if (m < pitch)  // kPreThreads threads: two rows at a time
            for (int r = 1 + (tid >> 7); r < kT && I * kT + r < L; r += 2)
                for (int cc = r; cc < kT && I * kT + cc < L; ++cc)
                    at[size_t(tri_row(L, I * kT + r, I * kT + cc)) * (pitch / 4)] = make_int4(int(kMark), int(kMark), int(kMark), int(kMark));
        return;
    }
    const int32_t* wa = ch.wa + size_t(b) * (L + 1);
    const int32_t* wd = ch.wdelta ? ch.wdelta + size_t(b) * (L + 1) : wa;
    const int t = tid + 1;
    const bool stage = t <= L;
    // a and delta of tensors t - 1 and t, the rest of stage t
    const int a_in = stage ? wa[t - 1] : 0, a_out = stage ? wa[t] : 0, d_out = stage ? wd[t] : 0;
    const int ab_in = stage ? ch.wabar[size_t(b) * L + t - 1] : 0;
    const int of_in = stage && ch.of ? ch.of[size_t(b) * L + t - 1] : 0, ob_in = stage && ch.ob ? ch.ob[size_t(b) * L + t - 1] : 0;
    const size_t words = tiles_of(L) * prog_words(pitch);  // progress and ticket words of a chain's tiles
    int32_t* prog = ws.prog + size_t(b) * words;
    const bool has_reach = flow && blocks_of(L) > 1;  // in the last of them
    __shared__ int s_part[kPreThreads / 64];

    if (part == parts) {  // once per chain
        __shared__ int s_flags[kPreThreads / 64], s_reach[kPreThreads / 64];
        const int f = stage ? ch.uf[size_t(b) * L + t - 1] : 0, bw = stage ? ch.ub[size_t(b) * L + t - 1] : 0;
        const int d_first = wd[0];
        if (b == 0 && tid == 0) ws.fault[0] = 0;
        int flags = 0;
        if (f < 0 || bw < 0) flags |= 1;
        if (f >= (1 << 30) || bw >= (1 << 30)) flags |= 2;
        for (int v : {a_in, a_out, d_out, d_first, ab_in, of_in, ob_in}) {  // a^0 and delta^0 among them
            if (v < 0) flags |= 1;
            if (v > (1 << 28)) flags |= 4;
        }
        if (ab_in < a_out) flags |= 8;  // abar^k must contain a^k: outside the Theorem's model
        const int fc = min(max(f, 0), (1 << 30) - 1), bc = min(max(bw, 0), 1 << 30);
        if (stage) {
            ws.fb[size_t(b) * L + t - 1] = int32_t(min(kInf, uint32_t(fc) + uint32_t(bc)));
            ws.wsh[size_t(b) * L + t - 1] = min(max(a_in, 0), pitch);
            ws.wabs[size_t(b) * L + t - 1] = min(max(ab_in, 0), pitch);
        }
        // prefix sums of the forward times, held at 2^30 (then the chain is flagged) and stored as 2^30 - 1
        auto held = [](int x, int y) { return int(min(uint32_t(x) + uint32_t(y), kInf)); };
        int sum = wave_scan(fc, held);
        // the largest shift; a^L is none
        const int reach = wave_scan(min(max(max(a_in, ab_in), 0), pitch), [](int x, int y) { return max(x, y); });
        flags = wave_scan(flags, [](int x, int y) { return x | y; });
        if (lane == 63) s_part[wave] = sum, s_flags[wave] = flags, s_reach[wave] = reach;
        __syncthreads();
        for (int w = 0; w < wave; ++w) sum = held(sum, s_part[w]);
        int32_t* P = ws.P + size_t(b) * (L + 1);
        if (tid == 0) P[0] = 0;
        if (stage) P[t] = min(sum, int(kInf) - 1);
        if (tid == int(blockDim.x) - 1) {  // the last thread's sum is the chain's
            int all = sum >= int(kInf) ? 2 : 0, most = 0;
            for (int w = 0; w <= wave; ++w) all |= s_flags[w], most = max(most, s_reach[w]);
            ws.flags[b] = all;
            if (has_reach) prog[words - 1] = most;
        }
        return;
    }

    for (size_t k = size_t(part) * blockDim.x + tid; k < words - (has_reach ? 1 : 0); k += size_t(parts) * blockDim.x) prog[k] = 0;
    // Sizes are clamped into [0, 2^28] so that thresholds of a bad chain cannot overflow.
    auto sz = [](int v) { return min(max(v, 0), 1 << 28); };
    const int a0 = sz(a_in), a1 = sz(a_out), d1 = sz(d_out), ab1 = sz(ab_in), f1 = sz(of_in), b1 = sz(ob_in);
    __shared__ int4 s_row[kPreThreads];  // what stage s brings to the thresholds of row s; w: what it needs where it lies between
    s_row[tid] = make_int4(ab1 + f1, d1 + ab1 + b1, a1 + f1, a0 + a1 + f1);
    const int s_lo = part * rows + 1, s_hi = min(s_lo + rows - 1, L);
    const int upto = wave_scan(stage && t > s_hi ? a0 + a1 + f1 : 0, [](int x, int y) { return max(x, y); });
    if (lane == 63) s_part[wave] = upto;
    int between = __shfl_up(upto, 1);  // largest of the stages s_hi + 1 .. t - 1
    if (lane == 0) between = 0;
    __syncthreads();
    for (int w = 0; w < wave; ++w) between = max(between, s_part[w]);
    for (int top = s_hi; top >= s_lo; top -= 4) {
        int4 row[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) row[u] = s_row[max(top - u, 1) - 1];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int s = top - u;
            if (s < s_lo) break;  // uniform
            if (s <= t && stage) {
                const int keep = max(d1 + row[u].x, row[u].y), ck = d1 + max(row[u].z, between);
                const size_t at = (size_t(b) * L + s - 1) * L + t - 1;
                ws.mall[at] = keep;
                ws.mnull[at] = ck;
                // A first, weak feasibility frontier: a finite cell passes at least one of its two gates.
                // The frontier kernel overwrites it with the exact one while the fill already runs;
                // whichever value a reader sees is a valid lower bound.
                ws.need[at] = min(keep, ck);
                if (s < t) between = max(between, row[u].w);
            }
        }
    }
}

// Feasibility frontier need[i][j] = smallest m at which cell (i, j) can be finite: the
// recurrence with costs dropped.  A leaf needs m_all; keeping abar^s needs
// max(m_all, omega_abar^s + need(s+1, t)); a checkpoint split at q needs
// max(m_null, omega_a^q + need(q, t), need(s, q-1)).  A cell below its frontier is infeasible
// whatever the times are, so the fill kernels skip work there.  Values saturate at 2^30,
// above any admissible M.  One block per chain, one segment length at a time; the triangle
// lives in LDS (row-major packed, L(L+1)/2 ints <= 127 KiB); 16 lanes share the splits of a cell.
__global__ void __launch_bounds__(1024) frontier_kernel(ckpt_chains_t ch, int L, Workspace ws) {
    const int b = blockIdx.x;
    const int tid = threadIdx.x;
    const int32_t* wa = ch.wa + size_t(b) * (L + 1);
    const int32_t* wab = ch.wabar + size_t(b) * L;
    auto sz = [](int v) { return min(max(v, 0), 1 << 28); };
    extern __shared__ int32_t s_need[];
    __shared__ int32_t s_wa[CKPT_MAX_L + 2];
    __shared__ int32_t s_wab[CKPT_MAX_L + 2];
    for (int k = tid; k <= L; k += blockDim.x) s_wa[k] = sz(wa[k]);
    for (int k = tid; k < L; k += blockDim.x) s_wab[k] = sz(wab[k]);
    int32_t* need = ws.need + size_t(b) * L * L;
    const int32_t* mallb = ws.mall + size_t(b) * L * L;
    const int32_t* mnullb = ws.mnull + size_t(b) * L * L;
    constexpr int kSat = 1 << 30;
    const int g = tid & 15, cells_per_pass = blockDim.x >> 4;
    __syncthreads();
    for (int d = 0; d < L; ++d) {
        for (int base = 0; base + d < L; base += cells_per_pass) {
            const int i = base + (tid >> 4), j = i + d;
            const bool valid = j < L;
            int split = kSat;
            int keep = 0, sweep = 0;
            if (valid && g == 0) keep = mallb[i * L + j], sweep = mnullb[i * L + j];  // in flight during the loop
            if (valid) {
                const int rowi = tri_row(L, i, i) - i;  // + j' = index of (i, j')
                for (int q = i + 1 + g; q <= j; q += 16)
                    split = min(split, max(min(kSat, s_wa[q] + s_need[tri_row(L, q, j)]), s_need[rowi + q - 1]));
            }
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) split = min(split, __shfl_xor(split, o));
            if (valid && g == 0) {
                int nd = keep;
                if (d > 0) {
                    const int opt_all = max(keep, min(kSat, s_wab[i] + s_need[tri_row(L, i + 1, j)]));
                    nd = min(opt_all, max(sweep, split));
                }
                nd = min(nd, kSat);
                s_need[tri_row(L, i, j)] = nd;
                need[i * L + j] = nd;
            }
        }
        __syncthreads();
    }
}

// Table reads go through a raw buffer descriptor of the chain's cost table: the address
// is descriptor base + per-lane byte offset (vector register, fixed for the whole kernel)
// + wave-uniform byte offset of the row (scalar register), so no vector instruction is
// spent on addressing, and a read outside the chain's table returns 0 instead of faulting.
// The scalar offset is 32-bit: a chain's table must stay below 4 GiB (checked on the host).
using rsrc_t = __amdgpu_buffer_rsrc_t;

__device__ __forceinline__ rsrc_t table_rsrc(const int32_t* tab, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(tab), 0, int(bytes), 0x00020000);
}

__device__ __forceinline__ uint32_t ld32(rsrc_t tab, uint32_t elem, uint32_t off) {
    return uint32_t(__builtin_amdgcn_raw_buffer_load_b32(tab, int(off), int(elem << 2), 0));
}

// Table accesses of the tile kernels: voff = per-lane byte offset (kNoRead: nothing is read, the
// result is 0), soff = wave-uniform byte offset.  dev = device scope.
__device__ __forceinline__ uint32_t tld(rsrc_t tab, uint32_t voff, uint32_t soff) {
    return uint32_t(__builtin_amdgcn_raw_buffer_load_b32(tab, int(voff), int(soff), 0));
}

// Orders a wave's LDS accesses before and after: its lanes read what other lanes of the wave wrote.
__device__ __forceinline__ void wave_settle() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wide accesses of a wave: eight rows of the table (the cells (i, jb) .. (i, jb + 7) of a row of a tile lie in consecutive
// ones), 64 columns each, as two instructions of 16 bytes a lane instead of eight of 4.  Lane l holds columns
// 4 (l & 15) .. + 3 of rows l >> 4 and 4 + (l >> 4); a turn through LDS brings values to lane = column, or from there.
// Fewer instructions, each whole lines: the compute unit's address path is busy 25 clocks a buffer instruction in the block product,
// 35 % of its time in 8 x 192 stages and 52 % in 64 x 96 (TA_TA_BUSY in profiles/): a share of the bound, not the bound.  Wide rows
// gained 0.4 to 1.1 % in large batches and nothing in small ones.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ u32x4 tld4(rsrc_t tab, uint32_t voff) {
    return __builtin_amdgcn_raw_buffer_load_b128(tab, int(voff), 0, 0);
}

// The only way to store 16 bytes a lane to a table: there is no scalar offset to give.  Behind a store of more than 8 bytes with a
// scalar offset register the compiler may write the first data register in the very next instruction, and the
// new value was seen in memory; without one it keeps them apart.
template <int policy>
__device__ __forceinline__ void tst4(rsrc_t tab, int voff, u32x4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(v, tab, voff, 0, policy);
}

constexpr int kPairs = kT * (kT - 1) / 2;  // splits in the column block of a row: (c2, cc), c2 < cc
__host__ __device__ constexpr int pair_index(int c2, int cc) { return c2 * (2 * kT - 1 - c2) / 2 + cc - c2 - 1; }

// Keeps the samples of cells (i, 8 J .. 8 J + 7): every kG-th lane stores its eight values.
__device__ __forceinline__ void store_samples(const Ctx& c, int b, int i, int J, uint32_t m, const uint32_t (&val)[kT]) {
    if (!c.ws.samp || (m & (kG - 1)) != kG - 1) return;
    int4* at = reinterpret_cast<int4*>(c.ws.samp + size_t(b) * samp_ints(c.L, c.pitch)) +
               2 * (size_t(4 * J * (J + 1) + i) * (c.pitch / kG) + m / kG);
    at[0] = make_int4(int(val[0]), int(val[1]), int(val[2]), int(val[3]));
    at[1] = make_int4(int(val[4]), int(val[5]), int(val[6]), int(val[7]));
}

// Which (chunk of m, tile, chain) a work-group takes.  The hardware hands work-groups out in
// linear order and to the 8 XCDs round-robin.  The linear index is re-read as (tile and chain)
// fastest, chunk slowest, so at every chunk level the tiles and chains spread evenly over the XCDs.
// rising: from the smallest budgets up.  Where the cells of a tile become feasible their upper bounds are infinite, and
// the chunks there keep 50 to 150 splits, others 4 to 16: in a launch of few work-groups they decide when it ends,
// so they start early, behind the ones below them that have nothing to do.  Launches of many work-groups (one slice)
// fill their tail with the cheap chunks at the low end: from the largest budget down.  Rising and falling: 3 x 254 stages,
// 1500 slots 2154 us and 2258, 20 x 80, 600 slots 425 and 429, 16 x 48, 1024 slots 211 and 216; with rising for one
// slice as well 64 x 96 stages, 2048 slots 3109 us and 3100, 8 x 192, 4096 slots 3681 and 3727.
struct Work { int chunk, tile, chain; };
__device__ __forceinline__ Work work_of_block(bool rising) {
    const uint32_t nt = gridDim.y * gridDim.z;
    const uint32_t lin = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const uint32_t level = lin / nt, t = lin - level * nt;
    return {int(rising ? level : gridDim.x - 1 - level), int(t % gridDim.y), int(t / gridDim.y)};
}

// + j = table row of cell (q, j)
__device__ __forceinline__ int row_base(int L, int q) { return q * L - (q * (q - 1)) / 2 - q; }

// Operands of the part of a row that does not depend on the row block: the splits in the
// column block (right operand (jb + c2 + 1, j) at its shift, for CF <= c2 < cc) and C_all (right
// operand (i + 1, j) at m - omega_abar^{i+1}).
template <int T, int CF>
__device__ __forceinline__ void load_row_tail(rsrc_t tab, const int32_t* __restrict__ wsh, int L, int pitch, int i,
                                              int jb, const int (&jc)[T], uint32_t wabi, uint32_t moff,
                                              uint32_t (&tj)[T][T], uint32_t (&al)[T]) {
#pragma unroll
    for (int cc = CF + 1; cc < T; ++cc)
#pragma unroll
        for (int c2 = CF; c2 < cc; ++c2) {
            const int q = min(jb + c2 + 1, L - 1);
            tj[c2][cc] = ld32(tab, uint32_t(row_base(L, q) + jc[cc]) * uint32_t(pitch) - uint32_t(wsh[q]), moff);
        }
#pragma unroll
    for (int cc = CF; cc < T; ++cc) {
        const int i1 = min(i + 1, L - 1);
        al[cc] = ld32(tab, uint32_t(row_base(L, i1) + max(jc[cc], i1)) * uint32_t(pitch) - wabi, moff);
    }
}

// Finishes the cells of row i in column block jb from the best candidate so far (splits in the
// row block, gemm partial): splits in the column block with the left operand (i, q-1) = the
// cell just finished, then the m_null gate, C_all with the m_all gate (smallest candidate
// number: wins ties), saturation, store.
template <int T, int CF, int DC>
__device__ __forceinline__ void finish_row(const Ctx& c, int b, size_t chain, const int32_t* __restrict__ P,
                                           const int32_t* __restrict__ mall, const int32_t* __restrict__ mnull,
                                           int L, int pitch, int i, int jb, int cend, const int (&jc)[T],
                                           uint32_t fbi, uint32_t m, uint32_t (&best)[T], uint32_t (&pick)[T],
                                           const uint32_t (&tj)[T][T], const uint32_t (&al)[T]) {
    const uint32_t Pi = P[i];
    const int rowi = tri_row(L, i, i) - i;  // + j = row of (i, j)
    uint32_t val[T];
#pragma unroll
    for (int cc = 0; cc < T; ++cc) val[cc] = kInf;
#pragma unroll
    for (int cc = CF; cc < T; ++cc) {
        const int j = jc[cc];
#pragma unroll
        for (int c2 = CF; c2 < cc; ++c2) {
            const int q = min(jb + c2 + 1, L - 1);  // left operand (i, q-1) = val[c2]
            const uint32_t v = val[c2] + (uint32_t(P[q]) - Pi) + tj[c2][cc];
            if (v < best[cc]) best[cc] = v, pick[cc] = q + 1;
        }
        const uint32_t ck = (m >= uint32_t(mnull[j])) ? min(best[cc], kInf) : kInf;
        uint32_t all = fbi;
        if (DC != 0 || cc > CF) all += al[cc];  // j > i
        all = (m >= uint32_t(mall[j])) ? min(all, kInf) : kInf;
        const bool take_all = all < kInf && all <= ck;
        const uint32_t fin = take_all ? all : ck;
        const uint32_t fpk = take_all ? uint32_t(i + 1) : (ck < kInf ? pick[cc] : 0u);
        val[cc] = fin;
        if (cc < cend) {
            const size_t o = chain + size_t(rowi + j) * pitch + m;
            c.cost[o] = int32_t(fin);
            c.arg[o] = uint8_t(fpk);
        }
    }
    store_samples(c, b, i, jb / T, m, val);
}

// Middle splits of every tile of block diagonal D >= 2, in two stages.
//
// Stage 1, bounds.  A cost never grows with m, so a cell's values at the two ends of a range of
// columns bound all values in between.  The fill keeps a sample of every cell at the last of every
// kG columns; from the samples below and above a sub-chunk of kG columns follow, for every cell of
// the tile and every split q, a lower bound of the candidate over the sub-chunk and an upper bound of
// the cell (the smallest upper bound of its candidates).  A split whose lower bound exceeds the upper
// bound in every cell and sub-chunk of the wave cannot attain any minimum and is dropped; ties stay.
// lane = (sub-chunk, split), 16 splits a pass; bounds are 32-bit sums of costs and prefix sums.
//
// Stage 2, candidates.  The splits that are left are evaluated for every cell and column, lane = m,
// as float64 keys  cost + (q+1)/256 : one add and one min per candidate give the minimum cost and,
// among equal costs, the smallest candidate number (all values are integers below 2^34 scaled by
// 2^-8, exact in float64; 2^44 is added so that cost and number stand in fixed bits of the mantissa).
//
// A wave owns 4 rows x 8 columns of cells for 64 columns of m; the two halves of a tile and CH
// adjacent chunks of m share a work-group (one half with four slices, see halves_of).
// Output, rows 0..6 of the tile: cost[] <- partial minimum clamped to 2^31 - 1, with bit 31 set as
// the mark "not finished", arg[] <- its number; the row kernels finish them.  Row 7 has no split
// in its own row block, so its partial minimum stays in registers and the wave finishes the row
// itself.
// What bounds it: the gathers of the samples and the chunks with the longest lists, 23 % of the vector issue
// slots busy; 2.2 ms a solve for L = 192, M = 4096, B = 8 at 4.5 TB/s asked for (2.5 and 4.6 with upper bounds from all splits), where evaluating every
// feasible split took 5.7 ms and 29 GB (5.5 % of the splits are left instead of 67 %).  kG = 16: bounds
// over 64 columns leave 11.7 %, over 32 7.5 %.  Half a tile a wave keeps it at 128 registers, four waves a SIMD.
// The epilogue reads nothing behind its stores (a load behind a store waits until it is through, and the
// compiler moves no load across a store to the tables): gates, shifts and prefix sums of row 7 are fetched
// with the splits at the start.  With scalar loads per column between the stores a launch took 2 to 4 us
// more (64 x 96 stages: 3.91 ms a solve with them, 3.51 without).  Rows go to the tables, and operands of row 7 come
// from them, as wide accesses through LDS: 3 stores a row instead of 16 and 9 loads instead of 36.
// KS > 1 (launches with too few tiles to fill the chip): KS waves share one half chunk, each takes
// every KS-th pass of stage 1 and every KS-th entry of the list, and their keys are merged
// through LDS at the end.
// Halves of a tile in one work-group.  The longest lists decide when a small launch ends, and evaluating them is float64
// issue: four slices of both halves would be two waves on every SIMD of one compute unit while others idle, so with four slices
// a half is a work-group of its own (1 x 254 stages, 1500 slots 1780 us with both, 1639 so; 1 x 128, 2048 slots 632 and 594;
// 1 x 192, 4096 slots 1192 and 1135; 3 x 254, 1500 slots 2205 and 2154).  Two slices fill the SIMDs once and keep both halves
// (3 x 254, 1500 slots 2154 us so, 2219 apart; but 8 x 128, 1024 slots 771 and 763, 16 x 48, 1024 slots 211 and 209).
constexpr int halves_of(int KS) { return KS >= 4 ? 1 : 2; }

template <int CH, int KS, bool CNT>
__global__ void __launch_bounds__(64 * halves_of(KS) * CH * KS, 4) gemm_kernel(Ctx c, int D) {
    constexpr int T = kT, R = T / 2, H = halves_of(KS);
    constexpr int NT = 64 * H * CH * KS;
    const Work w = work_of_block(KS > 1);
    const int b = c.b0 + w.chain, I = w.tile, J = I + D;
    const int L = c.L, pitch = c.pitch;
    const int qlo = (I + 1) * T, qhi = J * T;
    const int j0 = J * T;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int slice = wave % KS, half = H == 1 ? w.chunk & 1 : (wave / KS) & 1;
    const int grp = wave / KS;       // waves of one group share a list
    const int i0 = I * T + half * R;  // first row of this wave
    const int chunk = H == 1 ? w.chunk >> 1 : w.chunk * CH + wave / (2 * KS);  // this wave's 64 columns of m
    static_assert(H == 2 || CH == 1, "one chunk, one half");
    const uint32_t m = chunk * 64 + lane;
    const uint32_t moff = m * 4;
    const int cend = min(T, L - j0);
    const size_t chain = size_t(b) * c.rows * pitch;
    const rsrc_t tab = table_rsrc(c.cost + chain, uint32_t(c.rows) * uint32_t(pitch) * 4u);
    const rsrc_t atab = __builtin_amdgcn_make_buffer_rsrc(c.arg + chain, 0, int(uint32_t(c.rows) * uint32_t(pitch)), 0x00020000);
    const int32_t* need = c.ws.need + size_t(b) * L * L;
    const int32_t* P = c.ws.P + size_t(b) * (L + 1);

    __shared__ int2 s_split[CKPT_MAX_L + 2];              // shift and prefix sum of split qlo + k
    __shared__ int s_list[H * CH][CKPT_MAX_L + 2];        // the splits that are left: k = q - qlo
    __shared__ uint32_t s_ub[H * CH][4][R * T];           // upper bound of every cell in every sub-chunk
    __shared__ int s_n[H * CH];
    // row 7: gates of its cells, and prefix sums and (shifted) byte offsets of the right operands of the splits in the column block
    __shared__ int32_t s_mall[T], s_mnull[T], s_jP[T];
    __shared__ uint32_t s_pair[kPairs];
    __shared__ __align__(16) uint32_t s_turn[H * CH][T][64];  // a row of the tile on its way to lane = column or back
    __shared__ __align__(16) uint8_t s_num[H * CH][T][64];
    const int nq = qhi - qlo + 1;
    const int i7 = I * T + T - 1;
    if (threadIdx.x < T) {
        const int j = min(j0 + int(threadIdx.x), L - 1), q = min(j0 + int(threadIdx.x) + 1, L - 1);
        s_mall[threadIdx.x] = c.ws.mall[(size_t(b) * L + i7) * L + j];
        s_mnull[threadIdx.x] = c.ws.mnull[(size_t(b) * L + i7) * L + j];
        s_jP[threadIdx.x] = P[q];
    } else if (threadIdx.x >= 64 && threadIdx.x < 64 + T * T) {
        const int c2 = int(threadIdx.x - 64) >> 3, cc = threadIdx.x & 7, q = min(j0 + c2 + 1, L - 1);
        if (c2 < cc)
            s_pair[pair_index(c2, cc)] =
                cc < cend ? (uint32_t(row_base(L, q) + j0 + cc) * uint32_t(pitch) - uint32_t(c.ws.wsh[size_t(b) * L + q])) * 4u : kNoRead;
    }
    for (int k = threadIdx.x; k < nq; k += NT)
        s_split[k] = make_int2(c.ws.wsh[size_t(b) * L + qlo + k], P[qlo + k]);
    // A chunk below the frontier of every cell of the wave has no candidate.
    const bool active = chunk * 64 < pitch;
    int out_need = need[(i0 + ((lane >> 3) & (R - 1))) * L + min(j0 + (lane & 7), L - 1)];
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) out_need = min(out_need, __shfl_xor(out_need, o));
    const bool live7 = half == 1 && active && chunk * 64 + 63 >= __builtin_amdgcn_readlane(out_need, 8 * (R - 1));
#pragma unroll
    for (int o = 16; o > 4; o >>= 1) out_need = min(out_need, __shfl_xor(out_need, o));
    const bool search = active && chunk * 64 + 63 >= out_need;  // uniform over the waves of a group
    if (slice == 0) {
        for (int k = lane; k < 4 * R * T; k += 64) s_ub[grp][k >> 5][k & 31] = kInf - 1 + uint32_t(P[i0 + ((k & 31) >> 3)]);
        if (lane == 0) s_n[grp] = 0;
    }
    __syncthreads();

    if (c.ws.samp) {
        const int sub = lane >> 4, x = lane & 15;
        const int kk = chunk * 4 + sub;  // sub-chunk: columns kG kk .. kG kk + kG - 1
        const uint32_t line = uint32_t(pitch / kG) * 32u;  // bytes of the samples of a row of eight cells
        const rsrc_t smp = table_rsrc(c.ws.samp + size_t(b) * samp_ints(L, pitch), uint32_t(samp_rows(L)) * line);
        const uint32_t right0 = uint32_t(4 * J * (J + 1)) * line;
        struct Bound { uint32_t l[R], r[T]; };
        // Samples of cells (i0 + r, q - 1) at sampled column kl and (q, j0 + cc) at sampled column kr, plus
        // the prefix sum of q; infinite where the column does not exist.
        auto fetch = [&](Bound& v, int q, int kl, int kr) {
            const int jq = (q - 1) >> 3;
            const uint32_t lo = kl >= 0 ? uint32_t(4 * jq * (jq + 1) + i0) * line + uint32_t(kl) * 32u + uint32_t((q - 1) & 7) * 4u : kNoRead;
            const uint32_t ro = kr >= 0 ? right0 + uint32_t(q) * line + uint32_t(kr) * 32u : kNoRead;
#pragma unroll
            for (int r = 0; r < R; ++r) v.l[r] = uint32_t(__builtin_amdgcn_raw_buffer_load_b32(smp, int(lo), int(uint32_t(r) * line), 0));
            typedef uint32_t u4 __attribute__((ext_vector_type(4)));
            const u4 a = __builtin_amdgcn_raw_buffer_load_b128(smp, int(ro), 0, 0), d = __builtin_amdgcn_raw_buffer_load_b128(smp, int(ro), 16, 0);
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) v.r[cc] = a[cc], v.r[cc + 4] = d[cc];
        };
        auto settle = [&](Bound& v, uint32_t Pq, int kl, int kr) {
            if (kl < 0) {
#pragma unroll
                for (int r = 0; r < R; ++r) v.l[r] = kInf;
            }
#pragma unroll
            for (int cc = 0; cc < T; ++cc) v.r[cc] = (kr < 0 || cc >= cend ? kInf : v.r[cc]) + Pq;
        };
        const int passes = search ? (nq + 15) / 16 : 0;
        // upper bounds: left operand sampled at the column before the sub-chunk, right operand at the last
        // sampled column that the whole shifted sub-chunk lies above
        uint32_t ub[R][T];
        const int stride = 16 * KS;
        auto split_of = [&](int k0) { return min(k0 + x, nq - 1); };
        auto below = [&](int sh) { return ckpt_rules::right_below(kk, sh); };
        auto above = [&](int sh) { return ckpt_rules::right_above(kk, sh); };
        const int kend = passes * 16;
        // Any splits give an upper bound; the best ones are mostly those that finished neighbours took at the end of
        // the sub-chunk: the first row of the next tile down (8 cells), the last column of the tile to the left (4), and four
        // (the other slices: sixteen) spread over the range.  One pass instead of one for every 16 splits, and as many
        // splits are dropped: a pass is six loads, four of a word and two of 16 bytes, that gather about 30 lines.
        // With kAsk splits and fewer all are spread, which does without the trip to the neighbours' numbers (ckpt_rules.h).
        // 8 x 192 stages, 4096 slots: 4.00 -> 3.89 ms a solve; 3 x 254, 1500 slots: 2.39 -> 2.33.
        Bound nx;
        int2 sp;
        if (search) {
            int pick = ckpt_rules::spread_split(x, slice, KS, nq);
            if (slice == 0 && nq > ckpt_rules::kAsk && x < 12) {
                const int i8 = (I + 1) * T, row = x < 8 ? row_base(L, i8) + min(j0 + x, L - 1) : row_base(L, i0 + x - 8) + j0 - 1;
                pick = ckpt_rules::asked_split(x, int(__builtin_amdgcn_raw_buffer_load_b8(atab, row * pitch + kk * kG + kG - 1, 0, 0)), qlo, nq);
            }
            sp = s_split[pick];
            fetch(nx, qlo + pick, kk - 1, below(sp.x));
            settle(nx, uint32_t(sp.y), kk - 1, below(sp.x));
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int cc = 0; cc < T; ++cc) ub[r][cc] = nx.l[r] + nx.r[cc];
        }
        sp = s_split[split_of(slice * 16)];
        if (slice * 16 < kend) fetch(nx, qlo + split_of(slice * 16), kk, above(sp.x));
        __builtin_amdgcn_sched_barrier(0);
        if (search) {
            // minimum over the 16 lanes of a sub-chunk: two exchanges that halve the cells a lane holds, then
            // two rotations of the row of 16 lanes
            uint32_t h[R * T / 2], f[R * T / 4];
#pragma unroll
            for (int t = 0; t < R * T / 2; ++t) {
                const uint32_t e0 = ub[(2 * t) >> 3][(2 * t) & 7], e1 = ub[(2 * t + 1) >> 3][(2 * t + 1) & 7];
                const uint32_t mine = (x & 1) ? e1 : e0, other = (x & 1) ? e0 : e1;
                h[t] = min(mine, uint32_t(__builtin_amdgcn_update_dpp(0, int(other), 0xB1, 0xf, 0xf, true)));
            }
#pragma unroll
            for (int t = 0; t < R * T / 4; ++t) {
                const uint32_t mine = (x & 2) ? h[2 * t + 1] : h[2 * t], other = (x & 2) ? h[2 * t] : h[2 * t + 1];
                f[t] = min(mine, uint32_t(__builtin_amdgcn_update_dpp(0, int(other), 0x4E, 0xf, 0xf, true)));
                f[t] = min(f[t], uint32_t(__builtin_amdgcn_update_dpp(0, int(f[t]), 0x124, 0xf, 0xf, true)));
                f[t] = min(f[t], uint32_t(__builtin_amdgcn_update_dpp(0, int(f[t]), 0x128, 0xf, 0xf, true)));
                if (x < 4) atomicMin(&s_ub[grp][sub][4 * t + (x & 3)], f[t]);  // cell 4 t + 2 (x bit 1) + (x bit 0)
            }
        }
        if constexpr (KS > 1) __syncthreads();
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_sched_barrier(0);
        // lower bounds: left operand sampled at the last column of the sub-chunk, right operand at the first
        // sampled column that the whole shifted sub-chunk lies below
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int cc = 0; cc < T; ++cc) ub[r][cc] = s_ub[grp][sub][r * T + cc];
        for (int k0 = slice * 16; k0 < kend; k0 += stride) {
            Bound v = nx;
            const int2 cur = sp;
            sp = s_split[split_of(k0 + stride)];
            fetch(nx, qlo + split_of(k0 + stride), kk, above(sp.x));
            __builtin_amdgcn_sched_barrier(0);
            settle(v, uint32_t(cur.y), kk, above(cur.x));
            bool on = false;
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int cc = 0; cc < T; ++cc) on = on || v.l[r] + v.r[cc] <= ub[r][cc];
            unsigned long long mask = __ballot(on);
            mask |= mask >> 32;
            mask |= mask >> 16;
            const uint32_t bits = uint32_t(mask) & 0xffffu & ((1u << min(16, nq - k0)) - 1u);
            int at = 0;
            if (lane == 0) at = atomicAdd(&s_n[grp], __popc(bits));
            at = __builtin_amdgcn_readfirstlane(at);
            if (lane < 16 && (bits >> x & 1u)) s_list[grp][at + __popc(bits & ((1u << x) - 1u))] = k0 + x;
        }
        if (search) count_work<CNT>(c.work, 0, (R + 8) * (1u + unsigned(max(0, passes - slice + KS - 1) / KS)), 0);
    } else if (slice == 0 && search) {
        // No room for samples: the splits q for which some cell of the wave can have both operands feasible
        // somewhere in these 64 columns.
        const int m_hi = min(chunk * 64 + 63, pitch - 1);
        int n = 0;
        for (int base = 0; base < nq; base += 64) {
            const int k = base + lane, q = qlo + k;
            bool on = false;
            if (k < nq) {
                int tl = 1 << 30, tr = 1 << 30;
#pragma unroll
                for (int r = 0; r < R; ++r) tl = min(tl, need[(i0 + r) * L + q - 1]);
#pragma unroll
                for (int cc = 0; cc < T; ++cc) tr = min(tr, need[q * L + min(j0 + cc, L - 1)]);
                on = m_hi >= max(tl, tr + s_split[k].x);
            }
            const unsigned long long mask = __ballot(on);
            if (on) s_list[grp][n + __popcll(mask & ((1ull << lane) - 1ull))] = k;
            n += __popcll(mask);
        }
        if (lane == 0) s_n[grp] = n;
    }
    if constexpr (KS > 1) {
        __syncthreads();  // the other slices of the group read the list
    } else {
        if (!active) return;  // KS > 1: every wave stays for the barriers of the merge
        __builtin_amdgcn_wave_barrier();  // the wave reads what its own lanes wrote: LDS keeps a wave's order
        __builtin_amdgcn_sched_barrier(0);
    }
    // this wave's entries: slice, slice + KS, ...
    const int n_all = __builtin_amdgcn_readfirstlane(s_n[grp]);
    const int n = active && n_all > slice ? (n_all - slice + KS - 1) / KS : 0;

    // Addresses are descriptor + per-lane offset (the split's row, one add) + a scalar offset that stays for
    // the whole kernel: byte offsets of the wave's rows from row i0 and of the tile's columns from column j0.
    uint32_t rowstep[R], colstep[T];
#pragma unroll
    for (int r = 0; r < R; ++r) rowstep[r] = uint32_t(row_base(L, i0 + r) - row_base(L, i0)) * uint32_t(pitch) * 4u;
#pragma unroll
    for (int cc = 0; cc < T; ++cc) colstep[cc] = uint32_t(min(cc, L - 1 - j0)) * uint32_t(pitch) * 4u;
    const uint32_t left0 = uint32_t(row_base(L, i0) - 1);  // + q = row of (i0, q - 1)
    double key[R][T];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int cc = 0; cc < T; ++cc) key[r][cc] = kKeyBase + 4294967295.0;

    if (n > 0) {
        uint32_t buf[2][R + T];
        // Entries past the end of the list read nothing and count as infinite.
        auto load = [&](uint32_t(&v)[R + T], int t) {
            const int k = __builtin_amdgcn_readfirstlane(s_list[grp][slice + KS * min(t, n - 1)]);
            const int q = qlo + k;
            const uint32_t sh = uint32_t(__builtin_amdgcn_readfirstlane(s_split[k].x));
            const uint32_t left = t < n ? moff + (left0 + uint32_t(q)) * uint32_t(pitch) * 4u : kNoRead;
            const uint32_t right = t < n ? moff + (uint32_t(row_base(L, q) + j0) * uint32_t(pitch) - sh) * 4u : kNoRead;
#pragma unroll
            for (int r = 0; r < R; ++r) v[r] = tld(tab, left, rowstep[r]);
#pragma unroll
            for (int cc = 0; cc < T; ++cc) v[R + cc] = tld(tab, right, colstep[cc]);
        };
        auto compute = [&](const uint32_t(&v)[R + T], int t) {
            const int k = __builtin_amdgcn_readfirstlane(s_list[grp][slice + KS * min(t, n - 1)]);
            const double cq = t < n ? double(s_split[k].y) + double(qlo + k + 1) * (1.0 / 256.0) + kKeyBase : 2.0 * kKeyBase;
            double lk[R], rk[T];
#pragma unroll
            for (int r = 0; r < R; ++r) lk[r] = double(v[r]);
#pragma unroll
            for (int cc = 0; cc < T; ++cc) rk[cc] = double(v[R + cc]) + cq;
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int cc = 0; cc < T; ++cc) key[r][cc] = fmin(key[r][cc], lk[r] + rk[cc]);
        };
        // Straight-line bodies of two entries without branches, so that the loads of the next entry
        // are in flight while one is evaluated.
        load(buf[0], 0);
        for (int k = 0; k < n; k += 2) {
            load(buf[1], k + 1);
            __builtin_amdgcn_sched_barrier(0);
            compute(buf[0], k);
            __builtin_amdgcn_sched_barrier(0);
            load(buf[0], k + 2);
            __builtin_amdgcn_sched_barrier(0);
            compute(buf[1], k + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        count_work<CNT>(c.work, 0, unsigned(R + T) * unsigned(n), 0);
    }

    if constexpr (KS > 1) {
        // Merge: row by row, the waves of slices 1.. hand their keys to the wave of slice 0 through LDS.
        // Every wave of the work-group passes all barriers.
        __shared__ double s_red[H * CH][KS - 1][T][64];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (slice > 0) {
#pragma unroll
                for (int cc = 0; cc < T; ++cc) s_red[grp][slice - 1][cc][lane] = key[r][cc];
            }
            __syncthreads();
            if (slice == 0) {
#pragma unroll
                for (int o = 0; o < KS - 1; ++o)
#pragma unroll
                    for (int cc = 0; cc < T; ++cc) key[r][cc] = fmin(key[r][cc], s_red[grp][o][cc][lane]);
            }
            __syncthreads();
        }
        if (slice != 0 || !active) return;
    }

    // The mantissa of a key holds 256 cost + number: cost is the 32 bits from bit 8 on.
    auto partial = [&](int r, int cc, uint32_t Pi, uint32_t& cst, uint32_t& num) {
        const unsigned long long bits = __builtin_bit_cast(unsigned long long, key[r][cc]);
        cst = uint32_t(bits >> 8) - Pi;
        num = uint32_t(bits) & 255u;
    };
    // A partial minimum is stored with bit 31 set: a finished cell never exceeds 2^30, so whoever
    // reads the table can tell a cell that still waits for its row kernel from a finished one.
    // Partial minima of 2^31 - 1 and more are infeasible whatever they were and are clamped.
    uint32_t Pr[R];
#pragma unroll
    for (int r = 0; r < R; ++r) Pr[r] = uint32_t(P[i0 + r]);
    auto convert = [&](int r) {
#pragma unroll
        for (int cc = 0; cc < T; ++cc) {
            uint32_t cst, num;
            partial(r, cc, Pr[r], cst, num);
            s_turn[grp][cc][lane] = min(cst, 0x7fffffffu) | 0x80000000u;
            s_num[grp][cc][lane] = uint8_t(num);
        }
    };
    // The sliced variants have no room for the 36 registers of row 7's operands beside the keys of four rows: 16 were
    // spilled, a spill waited for the operands that had just been requested, and its reload stood behind the stores of the
    // rows.  With one row converted first nothing is spilled (123 registers): 1 x 192 stages, 4096 slots 1096 -> 1079 us, 3 x 254,
    // 1500 slots 2176 -> 2150, 8 x 96, 2048 slots 663 -> 653, 16 x 48, 1024 slots 213.1 -> 209.8.
    if constexpr (KS > 1) {
        convert(0);
        __builtin_amdgcn_sched_barrier(0);
    }

    // Row 7: operands of its column-block splits and of C_all are requested before the other rows
    // are converted and stored -- unless the whole chunk lies below the frontier of its cells.
    const int cell = lane >> 4, col = 4 * (lane & 15);
    const uint32_t wide = uint32_t(cell * pitch + chunk * 64 + col) * 4u;  // this lane's part of a wide access: row `cell` of eight
    u32x4 tjw[kPairs / 4], alw[2];
    uint32_t fb7 = 0;
    if (live7) {  // wave-uniform
#pragma unroll
        for (int k = 0; k < kPairs / 4; ++k) {
            const uint32_t at = s_pair[4 * k + cell];
            tjw[k] = tld4(tab, at == kNoRead ? kNoRead : at + uint32_t(chunk * 64 + col) * 4u);
        }
        fb7 = uint32_t(c.ws.fb[size_t(b) * L + i7]);
        const uint32_t below = wide + (uint32_t(row_base(L, i7 + 1) + j0) * uint32_t(pitch) - uint32_t(c.ws.wabs[size_t(b) * L + i7])) * 4u;
        alw[0] = tld4(tab, cell < cend ? below : kNoRead);
        alw[1] = tld4(tab, cell + 4 < cend ? below + 16u * uint32_t(pitch) : kNoRead);
    }
    // A row of the tile from s_turn and s_num to the tables.
    auto store_row = [&](int i) {
        wave_settle();
        const uint32_t at = wide + uint32_t(tri_row(L, i, j0)) * uint32_t(pitch) * 4u;
        const u32x4 lo = *reinterpret_cast<const u32x4*>(&s_turn[grp][cell][col]), hi = *reinterpret_cast<const u32x4*>(&s_turn[grp][cell + 4][col]);
        const u32x2 num = *reinterpret_cast<const u32x2*>(&s_num[grp][lane >> 3][8 * (lane & 7)]);
        const uint32_t at8 = uint32_t(tri_row(L, i, j0) + (lane >> 3)) * uint32_t(pitch) + uint32_t(chunk * 64 + 8 * (lane & 7));
        const int to_lo = int(cell < cend ? at : kNoRead), to_hi = int(cell + 4 < cend ? at + 16u * uint32_t(pitch) : kNoRead);
        const int to_num = int((lane >> 3) < cend ? at8 : kNoRead);
        auto put = [&](auto policy) {
            tst4<policy.value>(tab, to_lo, lo);
            tst4<policy.value>(tab, to_hi, hi);
            __builtin_amdgcn_raw_buffer_store_b64(num, atab, to_num, 0, policy.value);
        };
        if (KS == 1 && c.passing) put(std::integral_constant<int, 2>{});  // nontemporal
        else put(std::integral_constant<int, 0>{});
        wave_settle();
    };
    uint32_t best[T], pick[T];
    if (half == 1) {
#pragma unroll
        for (int cc = 0; cc < T; ++cc) partial(R - 1, cc, uint32_t(P[i7]), best[cc], pick[cc]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r == R - 1 && half == 1) break;  // row 7
        if (r > 0 || KS == 1) convert(r);
        store_row(i0 + r);
    }
    count_work<CNT>(c.work, 0, live7 ? 36u : 0u, unsigned(R) * unsigned(cend));
    if (half == 0) return;
    // splits in the column block with the left operand (i, q-1) = the cell just finished, then the m_null gate,
    // C_all with the m_all gate (smallest candidate number: wins ties), saturation
    uint32_t tj[kPairs], al[T], val[T];
    if (live7) {
        auto turn = [&](const u32x4& a, const u32x4& d) {
            *reinterpret_cast<u32x4*>(&s_turn[grp][cell][col]) = a;
            *reinterpret_cast<u32x4*>(&s_turn[grp][cell + 4][col]) = d;
            wave_settle();
        };
#pragma unroll
        for (int k = 0; k < kPairs; k += T) {
            turn(tjw[k / 4], k + 4 < kPairs ? tjw[min(k / 4 + 1, kPairs / 4 - 1)] : alw[0]);
#pragma unroll
            for (int u = 0; u < T; ++u) {
                if (k + u < kPairs) tj[k + u] = s_turn[grp][u][lane];
                else al[k + u - kPairs] = s_turn[grp][u][lane];
            }
            wave_settle();
        }
        static_assert(kPairs % T == 4, "the last turn holds four pairs and the first four operands of C_all");
        turn(alw[1], alw[1]);
#pragma unroll
        for (int u = 0; u < 4; ++u) al[4 + u] = s_turn[grp][u][lane];
        wave_settle();
    }
    const uint32_t Pi = Pr[R - 1];
#pragma unroll
    for (int cc = 0; cc < T; ++cc) {
        val[cc] = kInf;
        uint32_t num = 0;
        if (live7) {
#pragma unroll
            for (int c2 = 0; c2 < cc; ++c2) {
                const uint32_t v = val[c2] + (uint32_t(s_jP[c2]) - Pi) + tj[pair_index(c2, cc)];
                if (v < best[cc]) best[cc] = v, pick[cc] = min(j0 + c2 + 1, L - 1) + 1;
            }
            const uint32_t ck = (m >= uint32_t(s_mnull[cc])) ? min(best[cc], kInf) : kInf;
            const uint32_t all = (m >= uint32_t(s_mall[cc])) ? min(fb7 + al[cc], kInf) : kInf;
            const bool take_all = all < kInf && all <= ck;
            val[cc] = take_all ? all : ck;
            num = take_all ? uint32_t(i7 + 1) : (ck < kInf ? pick[cc] : 0u);
        }
        s_turn[grp][cc][lane] = val[cc];
        s_num[grp][cc][lane] = uint8_t(num);
    }
    store_row(i7);
    store_samples(c, b, i7, J, m, val);
}

// Finishes row R of every tile of block diagonal D: cells (i, j), i = I*T + R, j in block
// J = I + D.  One lane per m.  Candidate order = candidate number order, strict '<' keeps
// the smallest number among equal costs: near-i splits, gemm partial, near-j splits; C_all
// (number i + 1, the smallest) wins ties at the end.
// R and the diagonal class DC (0: D = 0, 1: D = 1, 2: D >= 2) are compile-time so that every
// trip count is static: all operand addresses are known up front, the loads are issued
// together and the kernel pays the memory latency once instead of once per split.
template <int T, int R, int DC>
__global__ void __launch_bounds__(kRowWG) row_kernel(Ctx c, int D) {
    constexpr int CF = (DC == 0) ? R : 0;                              // first column with j >= i
    constexpr int NQ = (DC == 0) ? 0 : (DC == 1 ? T - R : T - 1 - R);  // near-i splits (D = 1: and q = jb)
    constexpr int NQA = NQ > 0 ? NQ : 1;
    const Work w = work_of_block(false);
    const int b = c.b0 + w.chain, I = w.tile, J = I + D;
    const int L = c.L, pitch = c.pitch;
    const int i = I * T + R;
    if (i >= L) return;
    const uint32_t m = uint32_t(w.chunk) * kRowWG + threadIdx.x;
    if (m >= uint32_t(pitch)) return;
    const uint32_t moff = m * 4;
    const size_t chain = size_t(b) * c.rows * pitch;
    const rsrc_t tab = table_rsrc(c.cost + chain, uint32_t(c.rows) * uint32_t(pitch) * 4u);
    const int32_t* P = c.ws.P + size_t(b) * (L + 1);
    const int32_t* wsh = c.ws.wsh + size_t(b) * L;
    const int32_t* mall = c.ws.mall + (size_t(b) * L + i) * L;
    const int32_t* mnull = c.ws.mnull + (size_t(b) * L + i) * L;
    const int jb = J * T;
    const int cend = min(T, L - jb);  // columns of this tile that exist
    const uint32_t Pi = P[i];
    const uint32_t fbi = c.ws.fb[size_t(b) * L + i];
    const uint32_t wabi = c.ws.wabs[size_t(b) * L + i];
    const int rowi = tri_row(L, i, i) - i;  // + j = row of (i, j)
    auto rowq = [&](int q) { return row_base(L, q); };

    // Columns past the end of a ragged last block are computed on a clamped j and not stored.
    int jc[T];
#pragma unroll
    for (int cc = 0; cc < T; ++cc) jc[cc] = min(jb + cc, L - 1);

    // A wave whose whole chunk lies below the feasibility frontier of every cell of the row
    // stores "infeasible" and reads nothing.
    {
        // the frontier as far as it is known: the weak one of the precompute kernel (a finite cell
        // passes at least one of its two gates) until the frontier kernel has written the exact one
        const int32_t* need = c.ws.need + (size_t(b) * L + i) * L;
        int row_need = 1 << 30;
#pragma unroll
        for (int cc = CF; cc < T; ++cc)
            row_need = min(row_need, need[jc[cc]]);
        const int m_hi = __builtin_amdgcn_readfirstlane(int(m)) | 63;
        if (m_hi < row_need) {
#pragma unroll
            for (int cc = CF; cc < T; ++cc) {
                if (cc < cend) {
                    const size_t o = chain + size_t(rowi + jc[cc]) * pitch + m;
                    c.cost[o] = int32_t(kInf);
                    c.arg[o] = 0;
                }
            }
            uint32_t inf[T];
#pragma unroll
            for (int cc = 0; cc < T; ++cc) inf[cc] = kInf;
            store_samples(c, b, i, J, m, inf);
            return;
        }
    }

    // ---- every load of this row, issued before anything is consumed ----
    uint32_t nl[NQA], nr[NQA][T];   // near-i: left (i, q-1) and right (q, j) at m - omega_a^q
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int q = i + 1 + u;
        const uint32_t rq = uint32_t(rowq(q)), sh = uint32_t(wsh[q]);
        nl[u] = ld32(tab, uint32_t(rowi + q - 1) * uint32_t(pitch), moff);
#pragma unroll
        for (int cc = 0; cc < T; ++cc) nr[u][cc] = ld32(tab, (rq + jc[cc]) * uint32_t(pitch) - sh, moff);
    }
    uint32_t pc[T], pp[T];  // gemm partial
    if (DC == 2) {
#pragma unroll
        for (int cc = 0; cc < T; ++cc) {
            const size_t o = chain + size_t(rowi + jc[cc]) * pitch + m;
            pc[cc] = uint32_t(c.cost[o]) & 0x7fffffffu;  // bit 31 marks the gemm's partial minima
            pp[cc] = c.arg[o];
        }
    }
    uint32_t tj[T][T], al[T];
    load_row_tail<T, CF>(tab, wsh, L, pitch, i, jb, jc, wabi, moff, tj, al);

    // ---- evaluation ----
    uint32_t best[T], pick[T];
#pragma unroll
    for (int cc = 0; cc < T; ++cc) best[cc] = 0xffffffffu, pick[cc] = 0;
#pragma unroll
    for (int u = 0; u < NQ; ++u) {
        const int q = i + 1 + u;
        const uint32_t lb = nl[u] + (uint32_t(P[q]) - Pi);
#pragma unroll
        for (int cc = 0; cc < T; ++cc) {
            const uint32_t v = lb + nr[u][cc];
            if (v < best[cc]) best[cc] = v, pick[cc] = q + 1;
        }
    }
    if (DC == 2) {
#pragma unroll
        for (int cc = 0; cc < T; ++cc)
            if (pc[cc] < best[cc]) best[cc] = pc[cc], pick[cc] = pp[cc];
    }
    finish_row<T, CF, DC>(c, b, chain, P, mall, mnull, L, pitch, i, jb, cend, jc, fbi, m, best, pick, tj, al);
}

// ---------------------------------------------------------------------------
// All rows of every tile of one block diagonal in ONE launch.
//
// A work-group owns one band of kBand columns of m of one tile and finishes its rows bottom-up.
// Row r needs the row below it in the same tile at m - shift: from its own band, and from lower
// bands that other work-groups finish in the same launch.
//   - Inside the band the row below travels through LDS (two buffers, one barrier per row).
//   - Between bands it travels through memory.  The work-groups of a tile take its bands by ticket (an
//     atomic counter per tile: one counter for a whole launch made 800 work-groups queue for 5 us), in
//     ascending order, so whatever a wave waits for belongs to a work-group that already runs -- no
//     deadlock, whatever order the hardware starts work-groups in.
//     D >= 2: before its row is finished a cell holds the gemm's partial minimum, marked by bit 31
//     (finished cells never exceed 2^30), so a reader needs no flag and a writer never waits for
//     its stores: a lane that finds the mark simply reads again.  D < 2: the cells hold whatever
//     the caller's buffer held, so every wave publishes "rows finished" for its chunk of 64
//     columns once its stores of the row have completed, and readers wait for those flags
//     (looked at one row ahead of the need, while the wave waits for its own stores).
//     Every wait is bounded: when it expires the kernel sets the fault word and all work-groups
//     drain (ckpt_check_inputs then reports CKPT_E_INTERNAL).
// Coherence between compute units and between the L2 caches of the eight dies, without cache
// flushes: a cell of the table is written once per solve and only read after it was published.
// Finished rows are stored with device-scope stores (written through to memory before the
// store counts as complete) and rows of the same launch are read with device-scope loads
// (never served from a compute unit's L1 or from a stale line of another die's L2).  Lanes whose
// shifted column would be negative read nothing (an out-of-range buffer offset returns 0), so
// no line of the table is touched before its owner has written it.
// Each loaded operand of a split is kept in registers for all rows that use it: per tile and
// lane 7 x 8 + 28 + 64 operand loads instead of the 252 + 224 + 64 of one launch per row.
// What bounds it: the chain of row steps.  Loads and stores complete in issue order, so a load behind
// a row's stores waits until these are written through; what a row needs from earlier launches is
// therefore requested before the stores of the row below it, a wave asks memory for rows of
// this launch only where a shifted column lies below its band, and a number that the gemm already stored
// is not read and written again.  Both reads of the row below (operands of the splits, of C_all) are one round
// trip.  The rest of a step is issue: 900 instructions, so gates are selects on the operands, and what is
// the same for the whole wave is decided once.  5 chains of 53 stages: 26 us a launch, 34 us before; 334 -> 238 us
// a solve.
// ---------------------------------------------------------------------------
constexpr int kSpinLimit = 1 << 20;        // default polls of a wait before it gives up (seconds, never reached)


// Per-tile parameters of the row kernel, fetched once into LDS by the whole work-group: the
// rows' thresholds and frontier, prefix sums, shifts, and the byte offsets of the table rows the
// tile touches.  Inside the row steps nothing but table cells comes from memory, so a step
// costs one memory round trip, and an address is one add: every access is
// descriptor base + per-lane offset (row offset from here + 4 m - 4 shift) + cc * row pitch.
struct TilePar {
    int32_t mall[kT][kT], mnull[kT][kT];  // [r][cc]: cell (i0 + r, j_cc)
    int32_t need[kT];         // feasibility frontier of row r: the smallest of its cells
    int32_t Pi[kT + 1];       // P[i0 + u], u = 0..8
    int32_t Pj[kT];           // P[min(jb + c2 + 1, L - 1)]
    int32_t wsh[kT + 1];      // shift of split q = i0 + u
    int32_t wshj[kT];         // shift of split q = min(jb + c2 + 1, L - 1)
    uint32_t joff[kT];        // byte offset of cell (q, jb), the same q
    int32_t wabs[kT], fb[kT];
    uint32_t rowoff[kT + 1];  // byte offset of cell (i0 + u, jb) in the chain's cost table, u = 0..8
    uint32_t diagoff[kT];     // byte offset of cell (i0 + r, i0 + r)
};

template <int DC>
struct TileCtx {
    Ctx c;
    const TilePar* par;
    int b, I, J, L, pitch, i0, jb, cend, band;
    rsrc_t tab, atab;  // the chain's cost table (bytes) and candidate table
    uint32_t m, moff;
    uint32_t col4[kT];  // cc * pitch * 4: the scalar part of every address
    int32_t* prog;    // progress of this tile: [chunks of 64 columns]
    int chunk0;       // first chunk of this band
    int nwait;        // chunks below the band that this wave's shifted reads can reach
    int seen;         // lane k < nwait: progress of chunk chunk0 - 1 - k as last looked at
    bool dead;        // a wait expired: stop working, keep meeting the barriers (per wave)
    // right operands kept for all rows: ri[u][cc] = cell (i0 + u, j_cc) at m - omega_a^{i0+u}, u = 1..8
    // (rows of this tile; u = 8 is the first stage of the column block, D = 1 only);
    // rj[c2][cc] = cell (jb + c2 + 1, j_cc) at its shift, c2 < cc (column block, D >= 1)
    uint32_t ri[kT + 1][kT];
    uint32_t rj[kT][kT];
    // requested a row ahead: left operands (i, q-1) of the splits in the row block, gemm partials
    uint32_t nl[kT], pc[kT];
};

__device__ __forceinline__ uint32_t tld_dev(rsrc_t tab, uint32_t voff, uint32_t soff) {
    return uint32_t(__builtin_amdgcn_raw_buffer_load_b32(tab, int(voff), int(soff), 16));
}

// Requests the progress of the chunks below the band (lane k looks at chunk chunk0 - 1 - k);
// consumed by the next wait_rows_below, by which time the load has long returned.
template <int DC>
__device__ __forceinline__ void look_below(TileCtx<DC>& x) {
    const int k = threadIdx.x & 63;
    if (k < x.nwait) x.seen = __hip_atomic_load(x.prog + x.chunk0 - 1 - k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Every wave for itself: until each of the nwait chunks below the band has finished `rows` rows.
template <int DC>
__device__ __forceinline__ void wait_rows_below(TileCtx<DC>& x, int rows) {
    if (x.nwait == 0 || x.dead) return;
    const int lane = threadIdx.x & 63;
    bool ok = __all(lane >= x.nwait || x.seen >= rows) && x.nwait <= 64 && x.c.spin_limit >= 0;
    for (int spin = 0; !ok && spin < x.c.spin_limit; ++spin) {
        ok = true;
        for (int k = lane; k < x.nwait; k += 64)
            ok = ok && __hip_atomic_load(x.prog + x.chunk0 - 1 - k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= rows;
        ok = __all(ok);
        if (ok) break;
        if ((spin & 63) == 63 && __hip_atomic_load(x.c.ws.fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)
            break;
        __builtin_amdgcn_s_sleep(2);
    }
    if (!ok) {
        x.dead = true;
        if (lane == 0) __hip_atomic_store(x.c.ws.fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Cells (i0 + u, jb + cc), cc = first_cc .. cend - 1, of a row finished in THIS launch, at column m - sh (operands
// of the splits, out) and, if `both`, at column m - sh2 (operands of C_all, out2): from LDS if that column lies in
// this band (`below` = the row's buffer), else from the table with device-scope loads, in one round trip.
// D >= 2: the cells of the tile hold the gemm's partial minima, marked by bit 31, until their
// row is finished, so the read needs no flag: a lane that finds the mark reads again (bounded).
// D < 2: the caller has waited for the progress flags of the chunks that are read.
template <int DC, bool FULL, bool CNT>
__device__ __forceinline__ void read_row_below(TileCtx<DC>& x, const uint32_t (*below)[kBand], uint32_t rowoff, int first_cc,
                                               uint32_t sh, uint32_t (&out)[kT], bool both, uint32_t sh2, uint32_t (&out2)[kT]) {
    const int cend = FULL ? kT : x.cend;
    const int t = int(threadIdx.x) - int(sh), t2 = int(threadIdx.x) - int(sh2);  // columns inside the band
    const bool in_band = t >= 0, in_band2 = t2 >= 0;
    const bool far = !in_band && x.m >= sh, far2 = both && !in_band2 && x.m >= sh2;
#pragma unroll
    for (int cc = 0; cc < kT; ++cc) {
        if (cc >= first_cc && cc < cend) {
            out[cc] = below[cc][in_band ? t : 0];
            out2[cc] = below[cc][in_band2 ? t2 : 0];
        }
    }
    if (!__any(far || far2)) return;  // a wave whose shifted columns all lie in its band asks memory for nothing
    const uint32_t voff = far ? x.moff + rowoff - 4 * sh : kNoRead, voff2 = far2 ? x.moff + rowoff - 4 * sh2 : kNoRead;
    if (CNT && __any(far)) count_work<CNT>(x.c.work, 2, unsigned(max(0, cend - first_cc)), 0);
    if (CNT && __any(far2)) count_work<CNT>(x.c.work, 2, unsigned(max(0, cend - first_cc)), 0);
    uint32_t mem[kT], mem2[kT];
    auto fetch = [&]() {
        uint32_t marks = 0;
#pragma unroll
        for (int cc = 0; cc < kT; ++cc) {
            mem[cc] = mem2[cc] = 0;
            if (cc >= first_cc && cc < cend) mem[cc] = tld_dev(x.tab, voff, x.col4[cc]);  // only cells that exist
        }
#pragma unroll
        for (int cc = 0; cc < kT; ++cc)
            if (cc >= first_cc && cc < cend) mem2[cc] = tld_dev(x.tab, voff2, x.col4[cc]);
#pragma unroll
        for (int cc = 0; cc < kT; ++cc) marks |= mem[cc] | mem2[cc];
        return (marks >> 31) != 0;
    };
    bool again = fetch();
    if (DC == 2) {
        int spin = 0;
        if (x.c.spin_limit < 0) again = far || far2;  // forced: every read from another band gives up
        while (__any(again)) {  // some lane met a cell that its owner has not finished yet
            if (++spin > x.c.spin_limit ||
                ((spin & 63) == 0 && __hip_atomic_load(x.c.ws.fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                x.dead = true;
                if ((threadIdx.x & 63) == 0)
                    __hip_atomic_store(x.c.ws.fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_s_sleep(2);
            if (again) again = fetch();
        }
    }
#pragma unroll
    for (int cc = 0; cc < kT; ++cc) {
        if (cc >= first_cc && cc < cend) {
            out[cc] = in_band ? out[cc] : mem[cc];
            out2[cc] = in_band2 ? out2[cc] : mem2[cc];
        }
    }
}

// The number of a cell whose minimum is the gemm's partial: it stands in the table already.
constexpr uint32_t kKeepPick = 256;

// Requests what row R needs from earlier launches: left operands and the gemm's partial minima.
template <int DC, int R, bool FULL>
__device__ __forceinline__ void request_row(TileCtx<DC>& x) {
    constexpr int NQ = (DC == 0) ? 0 : (DC == 1 ? kT - R : kT - 1 - R);
    const TilePar& par = *x.par;
    const bool live = int(__builtin_amdgcn_readfirstlane(int(x.m)) | 63) >= par.need[R];  // else the row is infeasible in this chunk
    const uint32_t left = live ? x.moff + par.diagoff[R] : kNoRead;  // cell (i, i); (i, i + u) is u rows further
#pragma unroll
    for (int u = 0; u < NQ; ++u) x.nl[u] = tld(x.tab, left, x.col4[u]);
    if (DC == 2) {  // gemm partial; bit 31 marks it
        const int cend = FULL ? kT : x.cend;
        const uint32_t own = live ? x.moff + par.rowoff[R] : kNoRead;
#pragma unroll
        for (int cc = 0; cc < kT; ++cc) {
            if (cc < cend) x.pc[cc] = tld(x.tab, own, x.col4[cc]);
        }
    }
}

// FULL: the tile has all eight columns (always, except in the last column block of a chain whose
// length is not a multiple of eight); the tests for columns that do not exist then vanish.
template <int DC, int R, bool CNT, bool FULL>
__device__ __forceinline__ void tile_row(TileCtx<DC>& x, uint32_t (*s_row)[kT][kBand]) {
    constexpr int T = kT;
    constexpr int RF = (DC == 2) ? T - 2 : T - 1;                      // first row this kernel finishes
    constexpr int CF = (DC == 0) ? R : 0;                              // first column with j >= i
    constexpr int NQ = (DC == 0) ? 0 : (DC == 1 ? T - R : T - 1 - R);  // splits in the row block (D = 1: and q = jb)
    constexpr int U = R + 1;                                           // the row below
    const int L = x.L;
    const int cend = FULL ? T : x.cend;
    const int i = x.i0 + R;
    if (i >= L) return;  // ragged last block: uniform over the work-group
    const bool below_here = R < RF && i + 1 < L;  // the row below exists and belongs to this launch
    const uint32_t m = x.m, moff = x.moff;
    const TilePar& par = *x.par;
    const uint32_t (*below)[kBand] = s_row[U & 1];
    uint32_t (*mine)[kBand] = s_row[R & 1];
    uint32_t val[T];

    if (DC < 2 && below_here) wait_rows_below(x, RF - R);
    if (!x.dead) {
        const int m_hi = __builtin_amdgcn_readfirstlane(int(m)) | 63;
        const bool live = m_hi >= par.need[R];  // else the whole chunk lies below the feasibility frontier of the row
        const uint32_t wabi = par.wabs[R];
        uint32_t al[T];  // operands of C_all: cell (i + 1, j) at m - omega_abar^{i+1}, for j > i
        // ---- loads of this row, all issued together ----
        // the operands that the row below contributes to all rows above it, kept
        if ((U < T || DC == 1) && x.i0 + U < L) {
            const uint32_t sh = uint32_t(par.wsh[U]);
            if (below_here) {
                read_row_below<DC, FULL, CNT>(x, below, par.rowoff[U], DC == 0 ? U : 0, sh, x.ri[U], live, wabi, al);
            } else {  // finished by an earlier launch
                const uint32_t voff = m >= sh ? moff + par.rowoff[U] - 4 * sh : kNoRead;
#pragma unroll
                for (int cc = (DC == 0 ? U : 0); cc < T; ++cc)
                    if (cc < cend) x.ri[U][cc] = tld(x.tab, voff, x.col4[cc]);
            }
        }
        const unsigned cols = unsigned(max(0, cend - CF));  // cells of the row that exist
        // loads from earlier launches: the row below (first row of the kernel only), left operands, the
        // gemm's partial minima, C_all operands (first row only); reads of rows of this
        // launch are counted where they are issued, and only for waves that reach below their band
        count_work<CNT>(x.c.work, 2, (below_here ? 0u : cols) + (live ? unsigned(NQ) + (DC == 2 ? 8u : 0u) +
                                                                          (below_here ? 0u : cols) : 0u), cols);
        const uint32_t own = moff + par.rowoff[R];  // this lane's cell of the row, column block start
        if (live) {
            const uint32_t Pi = par.Pi[R];
            const uint32_t fbi = par.fb[R];
            if (!below_here && i + 1 < L) {  // row 0 of the tile below, or row 7 finished by the gemm: earlier launches
                const uint32_t voff = m >= wabi ? moff + par.rowoff[U] - 4 * wabi : kNoRead;
#pragma unroll
                for (int cc = (DC == 0 ? CF + 1 : CF); cc < T; ++cc)
                    if (cc < cend) al[cc] = tld(x.tab, voff, x.col4[cc]);
            }
            // ---- evaluation, in candidate-number order with strict '<' ----
            uint32_t best[T], pick[T];
#pragma unroll
            for (int u = 0; u < NQ; ++u) {
                const int q = i + 1 + u;
                const uint32_t lb = x.nl[u] + (uint32_t(par.Pi[R + 1 + u]) - Pi);
#pragma unroll
                for (int cc = 0; cc < T; ++cc) {
                    const uint32_t v = lb + x.ri[R + 1 + u][cc];
                    if (u == 0) best[cc] = v, pick[cc] = q + 1;
                    else if (v < best[cc]) best[cc] = v, pick[cc] = q + 1;
                }
            }
            if (DC == 2) {
#pragma unroll
                for (int cc = 0; cc < T; ++cc) {
                    const uint32_t v = x.pc[cc] & 0x7fffffffu;
                    if (cc < cend && v < best[cc]) best[cc] = v, pick[cc] = kKeepPick;
                }
            }
            // Before this row's stores are issued: a load that follows a store would wait until the store is written through.
            if constexpr (R > 0) request_row<DC, R - 1, FULL>(x);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int cc = CF; cc < T; ++cc) {
                if (NQ == 0) best[cc] = kInf, pick[cc] = 0;
#pragma unroll
                for (int c2 = CF; c2 < cc; ++c2) {  // splits in the column block: left operand (i, q-1) = val[c2]
                    const int q = min(x.jb + c2 + 1, L - 1);
                    const uint32_t r = (DC == 0) ? x.ri[c2 + 1][cc] : x.rj[c2][cc];
                    const uint32_t v = val[c2] + (uint32_t(par.Pj[c2]) - Pi) + r;
                    if (v < best[cc]) best[cc] = v, pick[cc] = q + 1;
                }
                // Gates; C_all has the smallest candidate number and wins ties.  Sums of 2^30 and more are infeasible
                // whatever they are.
                const uint32_t ck = m >= uint32_t(par.mnull[R][cc]) ? best[cc] : kInf;
                uint32_t all = m >= uint32_t(par.mall[R][cc]) ? fbi : kInf;
                if (DC != 0 || cc > CF) all += al[cc];  // j > i
                pick[cc] = all <= ck ? uint32_t(i + 1) : pick[cc];
                val[cc] = min(min(all, ck), kInf);
                pick[cc] = val[cc] < kInf ? pick[cc] : 0u;
            }
#pragma unroll
            for (int cc = CF; cc < T; ++cc) {
                if (cc < cend) {  // cost with a device-scope store: other bands read it in this launch
                    __builtin_amdgcn_raw_buffer_store_b32(int(val[cc]), x.tab, int(own), int(x.col4[cc]), 16);
                    const uint32_t at = DC == 2 && pick[cc] == kKeepPick ? kNoRead : own >> 2;
                    __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(pick[cc]), x.atab, int(at), int(x.col4[cc] >> 2), 0);
                }
            }
#pragma unroll
            for (int cc = 0; cc < CF; ++cc) val[cc] = kInf;  // no cells
        } else {
            if constexpr (R > 0) request_row<DC, R - 1, FULL>(x);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int cc = 0; cc < T; ++cc) val[cc] = kInf;
#pragma unroll
            for (int cc = CF; cc < T; ++cc) {
                if (cc < cend) {
                    __builtin_amdgcn_raw_buffer_store_b32(int(kInf), x.tab, int(own), int(x.col4[cc]), 16);
                    __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(0), x.atab, int(own >> 2), int(x.col4[cc] >> 2), 0);
                }
            }
        }
        store_samples(x.c, x.b, i, x.J, m, val);
        if (R > 0) {
            // the rows above read this row from LDS (this band) or from memory (bands above)
#pragma unroll
            for (int cc = CF; cc < T; ++cc) mine[cc][threadIdx.x] = val[cc];
            if (DC < 2) {
                // The cells of these tiles hold whatever the caller's buffer held: readers in other
                // bands need a flag.  Publish the row for this wave's chunk as soon as its stores
                // have completed; the look at the chunks below returns together with them.
                look_below(x);
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_s_waitcnt(0);
                if ((threadIdx.x & 63) == 0)
                    __hip_atomic_store(x.prog + (x.m >> 6), RF - R + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
    if (R > 0) __syncthreads();  // the row is in LDS for the waves of this band
}

template <int DC, int R, bool CNT, bool FULL>
struct TileRows {
    static __device__ __forceinline__ void run(TileCtx<DC>& x, uint32_t (*s_row)[kT][kBand]) {
        tile_row<DC, R, CNT, FULL>(x, s_row);
        if constexpr (R > 0) TileRows<DC, R - 1, CNT, FULL>::run(x, s_row);
    }
};

template <int DC, bool CNT>
__global__ void __launch_bounds__(kRowWG, 3) tile_rows_kernel(Ctx c, int D) {
    constexpr int T = kT;
    constexpr int RF = (DC == 2) ? T - 2 : T - 1;
    __shared__ int s_band, s_fault;
    __shared__ uint32_t s_row[2][kT][kBand];  // the last two finished rows of this band
    __shared__ TilePar s_par;
    // Work-groups are started in linear order: the first bands of all tiles and chains, then the second ones, ...
    const uint32_t items = gridDim.y * gridDim.z;
    const uint32_t item = (blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z)) % items;
    TileCtx<DC> x;
    x.c = c;
    x.I = int(item % gridDim.y);
    x.J = x.I + D;
    x.b = c.b0 + int(item / gridDim.y);
    x.prog = c.ws.prog + (size_t(x.b) * tiles_of(c.L) + tile_index(blocks_of(c.L), x.I, x.J)) * prog_words(c.pitch);
    if (threadIdx.x == kRowWG - 1) {  // a wave that fetches none of the parameters below
        s_band = atomicAdd(x.prog + c.pitch / 64, 1);
        s_fault = __hip_atomic_load(c.ws.fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    x.L = c.L;
    x.pitch = c.pitch;
    x.i0 = x.I * T;
    x.jb = x.J * T;
    x.cend = min(T, c.L - x.jb);
    const size_t chain = size_t(x.b) * c.rows * c.pitch;
    x.tab = table_rsrc(c.cost + chain, uint32_t(c.rows) * uint32_t(c.pitch) * 4u);
    x.atab = __builtin_amdgcn_make_buffer_rsrc(c.arg + chain, 0, int(uint32_t(c.rows) * uint32_t(c.pitch)), 0x00020000);
    x.seen = 0;
#pragma unroll
    for (int cc = 0; cc < T; ++cc) x.col4[cc] = uint32_t(cc) * uint32_t(c.pitch) * 4u;
#pragma unroll
    for (int u = 0; u <= T; ++u)
#pragma unroll
        for (int cc = 0; cc < T; ++cc) x.ri[u][cc] = 0;
#pragma unroll
    for (int c2 = 0; c2 < T; ++c2)
#pragma unroll
        for (int cc = 0; cc < T; ++cc) x.rj[c2][cc] = 0;
    const int32_t* P = c.ws.P + size_t(x.b) * (c.L + 1);
    const int32_t* wsh = c.ws.wsh + size_t(x.b) * c.L;
    {   // parameters of the tile: one fetch by the whole work-group
        const int t = threadIdx.x, L = c.L;
        const size_t bL = size_t(x.b) * L;
        if (t < 64) {
            const int r = t >> 3, i = min(x.i0 + r, L - 1);
            const size_t at = (bL + i) * L + min(x.jb + (t & 7), L - 1);  // no dynamic index into x: it stays in registers
            s_par.mall[r][t & 7] = c.ws.mall[at];
            s_par.mnull[r][t & 7] = c.ws.mnull[at];
            // weak or exact frontier, whichever is there: both are lower bounds
            int need = (t & 7) >= (DC == 0 ? r : 0) && (t & 7) < x.cend && x.i0 + r < L ? c.ws.need[at] : 1 << 30;
#pragma unroll
            for (int o = 4; o > 0; o >>= 1) need = min(need, __shfl_xor(need, o));
            if ((t & 7) == 0) s_par.need[r] = need;
        } else if (t < 64 + T + 1) {
            const int u = t - 64, q = min(x.i0 + u, L - 1);
            s_par.Pi[u] = P[min(x.i0 + u, L)];
            s_par.wsh[u] = wsh[q];
            // cell (q, jb); on the diagonal tile only the cells with jb + cc >= q exist and are touched
            s_par.rowoff[u] = uint32_t(row_base(L, q) + x.jb) * uint32_t(c.pitch) * 4u;
        } else if (t >= 96 && t < 96 + T) {
            const int r = t - 96, q = min(x.jb + r + 1, L - 1), i = min(x.i0 + r, L - 1);
            s_par.Pj[r] = P[q];
            s_par.wshj[r] = wsh[q];
            s_par.joff[r] = uint32_t(row_base(L, q) + x.jb) * uint32_t(c.pitch) * 4u;
            s_par.wabs[r] = c.ws.wabs[bL + i];
            s_par.fb[r] = c.ws.fb[bL + i];
            s_par.diagoff[r] = uint32_t(row_base(L, i) + i) * uint32_t(c.pitch) * 4u;
        }
    }
    x.par = &s_par;
    __syncthreads();
    x.band = __builtin_amdgcn_readfirstlane(s_band);
    if (x.band >= bands_of(c.pitch)) return;  // cannot happen: one ticket per work-group
    x.m = uint32_t(x.band) * kBand + threadIdx.x;
    x.moff = x.m * 4;
    x.dead = s_fault != 0;  // an earlier work-group gave up: drain
    {   // A band below the feasibility frontier of every cell this kernel finishes in the tile: all of
        // them are infeasible there.  Store that and leave (the whole work-group decides alike).
        int tile_need = 1 << 30;
#pragma unroll
        for (int r = 0; r <= RF; ++r) tile_need = min(tile_need, s_par.need[r]);
        if (int(min(uint32_t(x.band) * kBand + kBand - 1, uint32_t(c.pitch) - 1)) < tile_need) {
            unsigned cells = 0;
            if (x.m < uint32_t(c.pitch) && !x.dead) {
                for (int r = 0; r <= RF; ++r) {
                    if (x.i0 + r >= c.L) continue;
                    const uint32_t own = x.moff + s_par.rowoff[r];
                    for (int cc = (DC == 0 ? r : 0); cc < x.cend; ++cc) {  // no dynamic index into x: it stays in registers
                        const uint32_t col = uint32_t(cc) * uint32_t(c.pitch);
                        __builtin_amdgcn_raw_buffer_store_b32(int(kInf), x.tab, int(own), int(col * 4u), 16);
                        __builtin_amdgcn_raw_buffer_store_b8((unsigned char)(0), x.atab, int(own >> 2), int(col), 0);
                        ++cells;
                    }
                    uint32_t inf[T];
#pragma unroll
                    for (int cc = 0; cc < T; ++cc) inf[cc] = kInf;
                    store_samples(c, x.b, x.i0 + r, x.J, x.m, inf);
                }
                count_work<CNT>(c.work, 2, 0, cells);
                if (DC < 2) {  // readers in the bands above wait for this chunk's progress
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __builtin_amdgcn_s_waitcnt(0);
                    if ((threadIdx.x & 63) == 0)
                        __hip_atomic_store(x.prog + (x.m >> 6), RF + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            return;
        }
    }
    x.chunk0 = x.band * (kBand / 64);
    {   // chunks below the band that the shifts of this tile's rows can reach from this wave's columns
        int reach = 0;
        for (int r = 0; r < T; ++r) reach = max(reach, max(s_par.wsh[r], s_par.wabs[r]));
        const int m0 = __builtin_amdgcn_readfirstlane(int(x.m));  // first column of the wave
        x.nwait = max(0, x.chunk0 - (max(0, m0 - reach) >> 6));
    }
    // The band may lie past the end of the rows (pitch is a multiple of 64, not of kBand): those
    // waves read and store nothing but still meet every barrier.
    if (__builtin_amdgcn_readfirstlane(int(x.m)) >= c.pitch) {
        for (int r = RF; r > 0; --r)
            if (x.i0 + r < c.L) __syncthreads();
        return;
    }
#pragma unroll
    for (int cc = 0; cc < T; ++cc) x.nl[cc] = 0, x.pc[cc] = 0;
    if (DC >= 1 && !x.dead) {
        if (x.cend == T) request_row<DC, RF, true>(x);
        else request_row<DC, RF, false>(x);
        // operands of the splits in the column block, finished by earlier launches
#pragma unroll
        for (int c2 = 0; c2 < T - 1; ++c2) {
            const uint32_t sh = uint32_t(s_par.wshj[c2]);
            const uint32_t voff = x.m >= sh ? x.moff + s_par.joff[c2] - 4 * sh : kNoRead;
#pragma unroll
            for (int cc = c2 + 1; cc < T; ++cc)
                if (cc < x.cend) x.rj[c2][cc] = tld(x.tab, voff, x.col4[cc]);
        }
        count_work<CNT>(c.work, 2, 28u, 0);
    }
    if (x.cend == T)
        TileRows<DC, RF, CNT, true>::run(x, s_row);
    else
        TileRows<DC, RF, CNT, false>::run(x, s_row);
}

// ---------------------------------------------------------------------------
// Every tile of a solve in ONE launch (flow_kernel), for batches that leave the chip half empty.
//
// There a solve is a chain of dependent steps, and what it takes is the length of the chain: launches and the gaps between
// them, round trips to memory, and the instructions of a lone wave, 4.4 clocks a vector instruction and 8 a scalar one (measured; with
// four waves a SIMD the vector ones take 4.4 in all).  So a work-group owns one tile and 64 columns, and four lanes share a column.
//   - Splits between the blocks: the four waves fetch the 16 operand rows of a split together, 16 bytes a lane and two batches of
//     four splits ahead, and pass them through LDS; each evaluates 4 x 4 cells, lane = column, as float64 keys (see
//     gemm_kernel), about 500 clocks a split.  The partial minima stay in LDS.  BOUNDS: splits are dropped as in gemm_kernel, each
//     wave for four rows; the upper bounds of the splits whose operands the neighbours finish come from the minima found
//     so far.  Else all feasible ones are evaluated.
//   - Rows, bottom-up: a wave holds 16 columns, lane k of the four of a column cells k and k + 4 of the row.  A finished cell
//     reaches the other lanes of its column as the operand of an addition (quad broadcast).  A row is about 190 instructions, 1250 clocks,
//     where tile_rows_kernel takes 900, 5500 to 6500 clocks.
// No launch boundary separates the diagonals.
//   - A chain's work-groups take its tiles by ticket, in an order in which a tile stands behind all that it waits for (see
//     flow_place), so that belongs to work-groups that already run.  Every wait is bounded, see tile_rows_kernel.
//   - Rows of the same tile at columns below the band: every cell is marked by bit 31 until its row is finished, and a lane that
//     finds the mark reads again.  These reads are requested a row ahead, and mostly find the band below finished.
//     A tile's cells are marked by the work-group of the tile to its left, those of the first diagonal by precompute_kernel.
//   - Other tiles: a flag per tile and 64 columns, set behind its last store.  A tile waits for the tiles to its left and
//     below it, there at all chunks that the chain's largest shift can reach (upper bounds read samples up to 15 columns further
//     down: ckpt_rules::sample_chunks); those waited for theirs, so everything it
//     reads is finished.  The splits whose operands lie two diagonals down and more do not wait for the last one.
// Everything read is read with device scope: lines may lie in this die's L2 with the marks in them.
// Results bit for bit those of the other kernels.  us a solve, two launches a diagonal and this: 1 x 24 stages, 512 slots 67 and 37;
// 5 x 53, 777 slots 229 and 105; 16 x 48, 1024 slots 211 and 134; 10 x 50, 500 slots 214 and 94; 1 x 192, 4096 slots 1177 and 649; 3 x 254,
// 1500 slots 2273 and 1407 (the rule: ckpt_rules::flow_pays).
// What bounds it: of 26000 clocks a diagonal (5 x 53 stages) rows take 12000, the 16 splits of the last neighbours 8000 (500 each whether or
// not their operands are read from LDS ahead), their first operands 2300, the stores and the flag 2000.  By the counters (profiles/) a wave waits, for
// memory, LDS or the others, 67 % of that time, and vector issue fills 26 % of the chip.  Long chains fill the places for work-groups, four a
// compute unit, and then both count: 1 x 192 stages, a work-group takes 63000 clocks, of which a wave waits 54 %, in a queue to issue 19 %, and vector issue
// fills 55 % of the chip (3 x 254 stages 74000, 52, 22 and 60; 16 x 48 41000, 47, 21 and 56).
//
// Inside, a candidate of row i stands plus P[i]: a right operand carries the prefix sum of its split, and a split costs one addition.
// ---------------------------------------------------------------------------
template <class F, int... K>
__device__ __forceinline__ void for_each_of(std::integer_sequence<int, K...>, F&& f) {
    (f(std::integral_constant<int, K>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
    for_each_of(std::make_integer_sequence<int, N>{}, f);
}

// The value of lane K of every four lanes.
template <int K>
__device__ __forceinline__ uint32_t quad_lane(uint32_t v) {
    return uint32_t(__builtin_amdgcn_update_dpp(0, int(v), K * 0x55, 0xf, 0xf, true));
}

__device__ __forceinline__ u32x4 tld4_dev(rsrc_t tab, uint32_t voff) {
    return __builtin_amdgcn_raw_buffer_load_b128(tab, int(voff), 0, 16);
}

constexpr uint32_t kHuge = 0xbfffffffu;  // never smaller than a candidate that counts; no overflow on top of a cost
using ckpt_rules::kFar;                  // a byte offset beyond every row
constexpr int kFlow = 256;               // threads of a work-group: four waves, 64 columns of a tile
constexpr int kBatch = 4;                // splits whose operands pass through LDS together
constexpr int kLeft = kT * (kT + 1) / 2;

struct FlowRow {  // of row i = i0 + r; offsets and shifts in bytes
    int32_t sh, wab, Pu, fb;      // shift of split i + 1, of C_all; P[i + 1]; u_f + u_b
    int32_t P, under, own, need;  // P[i]; offsets of cells (i + 1, j0) and (i, j0); the row's frontier
};

template <bool BOUNDS>
struct FlowLds {
    static constexpr int NBUF = BOUNDS ? 1 : 2;
    union {
        uint32_t buf[NBUF][kBatch][2 * kT][64];  // operands of splits: left (i0 + r, q - 1), then right (q, j0 + cc) at its shift
        uint32_t stage[NBUF][64][64];            // the last: left operands of the row block, right operands of the column block
        struct {
            uint32_t part[kT * kT][64];       // partial minima plus P[i] and their numbers
            uint8_t pnum[kT * kT][64];
        } p;
    } u;
    uint32_t row[2][kT][72];
    __align__(16) uint8_t num[2][kT][64];
    int4 item[64];                            // staged rows: byte offset, shift, rotation of the columns in LDS
    int2 split[2][kFlow];                     // lists of splits: byte offset and shift of cell (i0, q - 1), of cell (q, j0)
    double key[kFlow];                        // P[q] + (q + 1) / 256 + kKeyBase
    FlowRow rows[kT];
    int4 gate[kT][4];                         // of cells k and k + 4: m_all, m_null
    int32_t Pj[kT];
    int32_t ticket, fault, reach, n_edge, n_inner;
};
struct FlowBounds {                           // bounds of the splits, see gemm_kernel
    int2 qp[kFlow];                           // of the lists: q, P[q]
    uint32_t ub[2][4][4 * kT];                // upper bound of every cell in every sub-chunk, rows 0 .. 3 and 4 .. 7
    uint8_t keep[2][kFlow];                   // which half of the rows needs an entry
    uint16_t index[kFlow];                    // the entries that are left, bits 8 and 9: for which half
    int32_t left;
};
constexpr int kEdge = 16;                     // the edge list: entries 0 .. 15, the inner list behind it

template <bool BOUNDS>
struct Flow {
    const Ctx& c;
    FlowLds<BOUNDS>& s;
    FlowBounds* bounds;
    rsrc_t tab, atab;
    int32_t* prog;
    int b, I, J, D, L, pitch, i0, j0, cend, m0, lane, wq;
    uint32_t rowpitch;
    size_t bl;
};

// The tile and band of a ticket.  Tiles are taken in the order of kSkew D + band, then of D, then of I: a band behind the one
// below it, a diagonal kSkew bands behind the last.  In the order of D alone neighbouring bands of a tile start together and
// wait for each other through all rows, 31000 clocks a tile instead of 12000, each holding its place on the chip; in the order of the
// bands alone diagonals do.  us a solve with 1, 3, 5, 8, 12, 24 and by D alone: 1 x 192 stages, 4096 slots 938, 747, 727, 738, 755, 805, 905;
// 3 x 254, 1500 slots 1562, 1583, 1620, 1662, 1703, 1818, 1818; 5 x 53, 777 slots 129, 118, 115, 113, 114, 114, 114.
constexpr int kSkew = 6;
struct FlowPlace { int D, band, I; };
__device__ __forceinline__ FlowPlace flow_place(int ticket, int nblk, int chunks, int lane) {
    // places before key k: of diagonals D < full all bands, of those up to `part` the bands below k - kSkew D
    auto before = [&](int k) {
        const int full = min(nblk, max(0, k - chunks + kSkew) / kSkew), part = min(nblk, (k + kSkew - 1) / kSkew);
        auto s1 = [](int n) { return n * (n - 1) / 2; };                // sums of D and D^2 below n
        auto s2 = [](int n) { return (n - 1) * n * (2 * n - 1) / 6; };
        return chunks * (full * nblk - s1(full)) + (part - full) * nblk * k - (k + kSkew * nblk) * (s1(part) - s1(full)) + kSkew * (s2(part) - s2(full));
    };
    // keys lie far below 64 * 64 (flow_pays): the last one with no more than `ticket` places before it
    int key = 64 * (__popcll(__ballot(before(64 * lane) <= ticket)) - 1);
    key += __popcll(__ballot(before(key + lane) <= ticket)) - 1;
    const int D0 = max(0, key - chunks + kSkew) / kSkew;  // first diagonal with this key
    ticket -= before(key);
    const int upto = lane * (nblk - D0) - lane * (lane - 1) / 2;  // places of `lane` diagonals from there
    const int n = __popcll(__ballot(D0 + lane <= nblk && upto <= ticket)) - 1;
    return {D0 + n, key - kSkew * (D0 + n), ticket - (n * (nblk - D0) - n * (n - 1) / 2)};
}

// Until the chunks chunk, chunk - 1, .. chunk - reach of both tiles are finished (first wave only).
template <bool BOUNDS>
__device__ __forceinline__ bool wait_tiles(const Flow<BOUNDS>& x, int tile_a, int tile_b, int chunk, int reach) {
    const int k = x.lane & 31, words = prog_words(x.pitch);
    const int32_t* flags = x.prog + size_t(x.lane < 32 ? tile_a : tile_b) * words + chunk;
    if (x.c.spin_limit < 0) return false;
    for (int base = 0; base <= min(reach, chunk); base += 32) {
        const int back = base + k;
        const bool look = back <= reach && back <= chunk;
        for (int spin = 0;; ++spin) {
            const bool ok = !look || __hip_atomic_load(flags - back, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0;
            if (__all(ok)) break;
            if (spin >= x.c.spin_limit ||
                ((spin & 63) == 63 && __hip_atomic_load(x.c.ws.fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0))
                return false;
            __builtin_amdgcn_s_sleep(1);
        }
    }
    return true;
}

// Marks this work-group's columns of rows 1 .. 7 of tile (I, J): what the waits inside that tile look for.
template <bool BOUNDS>
__device__ __forceinline__ void mark_tile(const Flow<BOUNDS>& x, int J) {
    const int cend = min(kT, x.L - J * kT);
    for (int s = x.wq; s < 14; s += 4) {  // four cells an instruction
        const int e = s * 4 + (x.lane >> 4), r = 1 + (e >> 3), cc = e & 7;
        const uint32_t at = (uint32_t(tri_row(x.L, x.i0 + r, J * kT + cc)) * uint32_t(x.pitch) + uint32_t(x.m0 + 4 * (x.lane & 15))) * 4u;
        tst4<16>(x.tab, int(cc < cend ? at : kNoRead), u32x4{kMark, kMark, kMark, kMark});
    }
}

// The rows of the tile, bottom-up.  DIAG: a tile of the first diagonal.
template <bool DIAG, bool BOUNDS>
__device__ __forceinline__ void flow_rows(Flow<BOUNDS>& x, const uint32_t (&leftL)[kT], const uint32_t (&leftH)[kT],
                                          const uint32_t (&colL)[kT], const uint32_t (&colH)[kT], uint32_t alL, uint32_t alH) {
    constexpr int T = kT, RF = T - 1;
    const Ctx& c = x.c;
    auto& s = x.s;
    const int lane = x.lane, k4 = lane & 3, cb = x.wq * 16 + (lane >> 2), cend = x.cend, L = x.L;
    const uint32_t rp = x.rowpitch;
    const int m = x.m0 + cb, cb4 = 4 * cb, below4 = 4 * x.m0;
    const int mine = (cb + 16 * k4) & 63;
    // this lane's cells from (row, j0); a cell that does not exist reads nothing
    const uint32_t ownL = uint32_t(k4) * rp, ownH = uint32_t(k4 + 4) * rp;
    const int mL4 = k4 < cend ? 4 * m : kFar, mH4 = k4 + 4 < cend ? 4 * m : kFar;
    // stores: two cells of 64 columns a wave, two columns a lane
    const int scell = 2 * x.wq + (lane >> 5), scol = 2 * (lane & 31);
    const uint32_t sown = uint32_t(scell) * rp + uint32_t(x.m0 + scol) * 4u;
    const bool sgo = scell < cend;
    // samples: the last column of a wave is the last of a sub-chunk
    const uint32_t line = uint32_t(x.pitch / kG) * uint32_t(4 * T);
    const rsrc_t smp = table_rsrc(c.ws.samp + (BOUNDS ? size_t(x.b) * samp_ints(L, x.pitch) : 0), BOUNDS ? uint32_t(samp_rows(L)) * line : 0);
    const uint32_t sat = (lane >> 2) == 15 ? uint32_t(4 * x.J * (x.J + 1) + x.i0) * line + uint32_t(m / kG) * uint32_t(4 * T) + 4u * uint32_t(k4) : kNoRead;

    uint32_t below[T + 1][2];
#pragma unroll
    for (int u = 0; u <= T; ++u) below[u][0] = below[u][1] = kHuge;
    uint32_t pf[4] = {0, 0, 0, 0}, po[4] = {kNoRead, kNoRead, kNoRead, kNoRead};  // operands from lower bands, requested a row ahead, and where
    auto fetch = [&]() {
        pf[0] = tld_dev(x.tab, po[0], 0), pf[1] = tld_dev(x.tab, po[1], 0);
        pf[2] = tld_dev(x.tab, po[2], 0), pf[3] = tld_dev(x.tab, po[3], 0);
    };
    FlowRow now = s.rows[RF];
    unrolled<RF + 1>([&](auto step) {
        constexpr int R = RF - decltype(step)::value, U = R + 1, CF = DIAG ? R : 0;
        const FlowRow w = now;
        if constexpr (R > 0) now = s.rows[R - 1];
        if (DIAG && x.i0 + R >= L) return;  // ragged last block: uniform over the work-group
        uint32_t bL = 0xffffffffu, bH = 0xffffffffu, nL = 0, nH = 0;
        if constexpr (!DIAG) {
            bL = s.u.p.part[R * T + k4][mine], bH = s.u.p.part[R * T + k4 + 4][mine];
            nL = s.u.p.pnum[R * T + k4][mine], nH = s.u.p.pnum[R * T + k4 + 4][mine];
        }
        const int4 gate = s.gate[R][k4];
        if constexpr (R < RF) {
            const int t = max(cb4 - w.sh, 0), t2 = max(cb4 - w.wab, 0);
            const char* row = reinterpret_cast<const char*>(&s.row[U & 1][k4][0]);
            constexpr int hi = 4 * 72 * 4;
            uint32_t rL = *reinterpret_cast<const uint32_t*>(row + t), rH = *reinterpret_cast<const uint32_t*>(row + t + hi);
            alL = *reinterpret_cast<const uint32_t*>(row + t2), alH = *reinterpret_cast<const uint32_t*>(row + t2 + hi);
            bool again = int(pf[0] | pf[1] | pf[2] | pf[3]) < 0;
            if (c.spin_limit < 0) again = (po[0] & po[1] & po[2] & po[3]) != kNoRead;  // forced: every read from another band gives up
            if (__any(again)) {  // some lane met a cell that its owner has not finished yet
                for (int spin = 0; __any(again); ++spin) {
                    if (spin >= c.spin_limit ||
                        ((spin & 63) == 63 && __hip_atomic_load(c.ws.fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                        if (lane == 0) __hip_atomic_store(c.ws.fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        break;
                    }
                    if (again) {
                        fetch();
                        again = int(pf[0] | pf[1] | pf[2] | pf[3]) < 0;
                    }
                }
            }
            const bool out = cb4 < w.sh, out2 = cb4 < w.wab;
            rL = (out ? pf[0] : rL) + uint32_t(w.Pu), rH = (out ? pf[1] : rH) + uint32_t(w.Pu);
            alL = out2 ? pf[2] : alL, alH = out2 ? pf[3] : alH;
            if constexpr (DIAG) {
                rL = k4 >= U && x.i0 + U < L ? rL : kHuge;
                rH = k4 + 4 >= U && x.i0 + U < L ? rH : kHuge;
            }
            below[U][0] = rL, below[U][1] = rH;
        }
        if constexpr (R > 0) {  // the next row's operands from the bands below: mostly finished there already
            auto far = [&](int m4, uint32_t own, int shift, bool exists) {  // columns below the band, not below zero
                const uint32_t e = uint32_t(m4 - shift);
                return exists && e < uint32_t(below4) ? own + uint32_t(now.under) + e : kNoRead;
            };
            const bool isL = !DIAG || k4 >= R, isH = !DIAG || k4 + 4 >= R;
            po[0] = far(mL4, ownL, now.sh, isL), po[1] = far(mH4, ownH, now.sh, isH);
            po[2] = far(mL4, ownL, now.wab, isL), po[3] = far(mH4, ownH, now.wab, isH);
            fetch();
        }
        // splits of the row block, in falling order with <=: the smallest number among equal costs stays
        if constexpr (!DIAG)
            unrolled<T - 1>([&](auto up) {
                constexpr int v = T - 2 - decltype(up)::value;  // left operand (i, i0 + v), split i0 + v + 1
                if constexpr (v >= R) {
                    const uint32_t l = v < 4 ? quad_lane<v & 3>(leftL[R]) : quad_lane<v & 3>(leftH[R]);
                    const uint32_t a = l + below[v + 1][0], d = l + below[v + 1][1];
                    const uint32_t q = uint32_t(x.i0 + v + 2);
                    nL = a <= bL ? q : nL, bL = min(a, bL);
                    nH = d <= bH ? q : nH, bH = min(d, bH);
                }
            });
        // gates: a closed one is larger than any candidate
        const uint32_t ckL = uint32_t((m - gate.y) >> 31), ckH = uint32_t((m - gate.w) >> 31);
        uint32_t aL = alL, aH = alH;
        if constexpr (DIAG) {  // a chain of one stage
            if (k4 == R) aL = 0;
            if (k4 + 4 == R) aH = 0;
        }
        aL = (uint32_t(w.fb) + aL) | uint32_t((m - gate.x) >> 31);
        aH = (uint32_t(w.fb) + aH) | uint32_t((m - gate.z) >> 31);
        const uint32_t p = uint32_t(w.P);
        unrolled<T - 1>([&](auto c2c) {  // splits of the column block: left operand = the cell just finished
            constexpr int c2 = decltype(c2c)::value;
            if constexpr (c2 >= CF) {
                const uint32_t v = c2 < 4 ? min(min(aL, max(bL - p, ckL)), kInf) : min(min(aH, max(bH - p, ckH)), kInf);
                const uint32_t l = quad_lane<c2 & 3>(v);
                const uint32_t q = uint32_t(x.j0 + c2 + 2);
                if constexpr (c2 < 3) {
                    const uint32_t a = l + (DIAG ? below[c2 + 1][0] : colL[c2]);
                    nL = a < bL ? q : nL, bL = min(a, bL);
                }
                const uint32_t d = l + (DIAG ? below[c2 + 1][1] : colH[c2]);
                nH = d < bH ? q : nH, bH = min(d, bH);
            }
        });
        const uint32_t cL = max(bL - p, ckL), cH = max(bH - p, ckH);
        const uint32_t vL = min(min(aL, cL), kInf), vH = min(min(aH, cH), kInf);
        nL = aL <= cL ? uint32_t(x.i0 + R + 1) : nL, nH = aH <= cH ? uint32_t(x.i0 + R + 1) : nH;
        nL = vL < kInf ? nL : 0u, nH = vH < kInf ? nH : 0u;
        s.row[R & 1][k4][cb] = vL, s.row[R & 1][k4 + 4][cb] = vH;
        s.num[R & 1][k4][cb] = uint8_t(nL), s.num[R & 1][k4 + 4][cb] = uint8_t(nH);
        if constexpr (BOUNDS) {
            __builtin_amdgcn_raw_buffer_store_b32(int(vL), smp, int(sat), int(R * line), 16);
            __builtin_amdgcn_raw_buffer_store_b32(int(vH), smp, int(sat), int(R * line + 16), 16);
        }
        __syncthreads();
        {   // without a branch: the next row's wait for its operands can then tell these stores from them
            const u32x2 v = *reinterpret_cast<const u32x2*>(&s.row[R & 1][scell][scol]);
            const uint16_t n = *reinterpret_cast<const uint16_t*>(&s.num[R & 1][scell][scol]);
            const uint32_t at = sown + uint32_t(w.own);
            const bool go = sgo && (!DIAG || scell >= CF);
            __builtin_amdgcn_raw_buffer_store_b64(v, x.tab, int(go ? at : kNoRead), 0, 16);
            __builtin_amdgcn_raw_buffer_store_b16(n, x.atab, int(go ? at >> 2 : kNoRead), 0, 0);
        }
    });
}

// Puts the splits q of 64 lanes that can be feasible in these columns into a list in LDS (one wave; the order does not matter).
__device__ __forceinline__ void list_splits(const Flow<false>& x, int q, bool valid, int first, int32_t* count) {
    const Ctx& c = x.c;
    auto& s = x.s;
    const int L = x.L;
    const int32_t* need = c.ws.need + x.bl * L;
    const int sh = c.ws.wsh[x.bl + q], P = c.ws.P[size_t(x.b) * (L + 1) + q];
    int tl = 1 << 30, tr = 1 << 30;
#pragma unroll
    for (int r = 0; r < kT; ++r) {
        tl = min(tl, need[(x.i0 + r) * L + q - 1]);
        tr = min(tr, need[q * L + min(x.j0 + r, L - 1)]);
    }
    const bool on = valid && x.m0 + 63 >= max(tl, tr + sh);
    const unsigned long long mask = __ballot(on);
    int at = 0;
    if (x.lane == 0) at = atomicAdd(count, __popcll(mask));
    at = first + __builtin_amdgcn_readfirstlane(at) + __popcll(mask & ((1ull << x.lane) - 1ull));
    if (on) {
        s.split[0][at] = make_int2(int(uint32_t(row_base(L, x.i0) + q - 1) * x.rowpitch), 0);
        s.split[1][at] = make_int2(int(uint32_t(row_base(L, q) + x.j0) * x.rowpitch), 4 * sh);
        s.key[at] = double(P) + double(q + 1) * (1.0 / 256.0) + kKeyBase;
    }
}

// Bounds of sixteen splits at the four sub-chunks of the band, for four rows: lane = (sub-chunk, split).
struct FlowBound { uint32_t l[kT / 2], r[kT]; };
__device__ __forceinline__ void fetch_bound(const Flow<true>& x, rsrc_t smp, FlowBound& v, int q, int half, int kl, int kr) {
    const uint32_t line = uint32_t(x.pitch / kG) * uint32_t(4 * kT);
    const int jq = (q - 1) >> 3;
    const uint32_t lo = kl >= 0 ? uint32_t(4 * jq * (jq + 1) + x.i0 + 4 * half) * line + uint32_t(kl) * uint32_t(4 * kT) + uint32_t((q - 1) & 7) * 4u : kNoRead;
    const uint32_t ro = kr >= 0 ? uint32_t(4 * x.J * (x.J + 1) + q) * line + uint32_t(kr) * uint32_t(4 * kT) : kNoRead;
#pragma unroll
    for (int r = 0; r < kT / 2; ++r) v.l[r] = tld_dev(smp, lo, uint32_t(r) * line);
    const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(smp, int(ro), 0, 16), d = __builtin_amdgcn_raw_buffer_load_b128(smp, int(ro), 16, 16);
#pragma unroll
    for (int cc = 0; cc < 4; ++cc) v.r[cc] = a[cc], v.r[cc + 4] = d[cc];
}
__device__ __forceinline__ void settle_bound(const Flow<true>& x, FlowBound& v, uint32_t Pq, int kl, int kr) {
#pragma unroll
    for (int r = 0; r < kT / 2; ++r) v.l[r] = kl < 0 ? kInf : v.l[r];
#pragma unroll
    for (int cc = 0; cc < kT; ++cc) v.r[cc] = (kr < 0 || cc >= x.cend ? kInf : v.r[cc]) + Pq;
}

// Upper bounds of the cells from 32 splits spread over a list of n (first .. first + n - 1), 16 a wave.
__device__ __forceinline__ void upper_bounds(Flow<true>& x, rsrc_t smp, int first, int n) {
    constexpr int R = kT / 2, T = kT;
    const int half = x.wq & 1, slice = x.wq >> 1, sub = x.lane >> 4, v = x.lane & 15, kk = x.m0 / kG + sub;
    const int e = first + (2 * (16 * slice + v) + 1) * n / 64;
    const int2 qp = x.bounds->qp[e];
    const int kl = ckpt_rules::left_below(kk), kr = ckpt_rules::right_below(kk, x.s.split[1][e].y >> 2);
    FlowBound w;
    fetch_bound(x, smp, w, qp.x, half, kl, kr);
    settle_bound(x, w, uint32_t(qp.y), kl, kr);
    // minimum over the 16 lanes of a sub-chunk, as in gemm_kernel
    uint32_t h[R * T / 2];
#pragma unroll
    for (int t = 0; t < R * T / 2; ++t) {
        const uint32_t e0 = w.l[(2 * t) >> 3] + w.r[(2 * t) & 7], e1 = w.l[(2 * t + 1) >> 3] + w.r[(2 * t + 1) & 7];
        const uint32_t mine = (v & 1) ? e1 : e0, other = (v & 1) ? e0 : e1;
        h[t] = min(mine, uint32_t(__builtin_amdgcn_update_dpp(0, int(other), 0xB1, 0xf, 0xf, true)));
    }
#pragma unroll
    for (int t = 0; t < R * T / 4; ++t) {
        const uint32_t mine = (v & 2) ? h[2 * t + 1] : h[2 * t], other = (v & 2) ? h[2 * t] : h[2 * t + 1];
        uint32_t f = min(mine, uint32_t(__builtin_amdgcn_update_dpp(0, int(other), 0x4E, 0xf, 0xf, true)));
        f = min(f, uint32_t(__builtin_amdgcn_update_dpp(0, int(f), 0x124, 0xf, 0xf, true)));
        f = min(f, uint32_t(__builtin_amdgcn_update_dpp(0, int(f), 0x128, 0xf, 0xf, true)));
        if (v < 4) atomicMin(&x.bounds->ub[half][sub][4 * t + (v & 3)], f);
    }
}

// Splits 16 p + slice .. of a list that can attain a minimum of four rows: their lower bound is at most the upper bound of some cell in
// some sub-chunk.  Every entry's answer is written, by the wave of its half.
// `between` runs behind the first request and ends in a barrier.
template <int SLICES, class F>
__device__ __forceinline__ void lower_bounds(Flow<true>& x, rsrc_t smp, int first, int n, F&& between) {
    constexpr int T = kT, R = T / 2;
    const int half = x.wq & 1, slice = x.wq >> 1, sub = x.lane >> 4, v = x.lane & 15, kk = x.m0 / kG + sub;
    FlowBound next;
    int2 qp;
    int kr = 0;
    auto request = [&](int k) {
        const int e = first + min(k + v, n - 1);
        qp = x.bounds->qp[e];
        kr = ckpt_rules::right_above(kk, x.s.split[1][e].y >> 2);
        fetch_bound(x, smp, next, qp.x, half, ckpt_rules::left_above(kk), kr);
    };
    if (slice < SLICES) request(16 * slice);
    between();
    if (slice >= SLICES) return;
    uint32_t ub[R][T];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int cc = 0; cc < T; ++cc) ub[r][cc] = x.bounds->ub[half][sub][r * T + cc];
    for (int k = 16 * slice; k < n; k += 16 * SLICES) {
        FlowBound w = next;
        const uint32_t Pq = uint32_t(qp.y);
        const int kc = kr;
        if (k + 16 * SLICES < n) request(k + 16 * SLICES);
        settle_bound(x, w, Pq, ckpt_rules::left_above(kk), kc);
        // a left operand not above ub - right for some column; nothing above zero is lost where the difference would be negative
        bool on = false;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            uint32_t most = 0;
#pragma unroll
            for (int cc = 0; cc < T; ++cc) most = max(most, __builtin_elementwise_sub_sat(ub[r][cc], w.r[cc]));
            on = on || w.l[r] <= most;
        }
        unsigned long long mask = __ballot(on);
        mask |= mask >> 32;
        mask |= mask >> 16;
        if (x.lane < 16 && k + v < n) x.bounds->keep[half][first + k + v] = uint8_t(uint32_t(mask) >> v & 1u);
    }
}

// The entries of a list that some half of the rows needs, into bounds->index.  Every wave, behind a barrier; ends in one.
__device__ __forceinline__ int left_over(Flow<true>& x, int first, int n, bool all) {
    const int t = threadIdx.x;
    const uint32_t f = t >= n ? 0u : all ? 3u : uint32_t(x.bounds->keep[0][first + t]) | uint32_t(x.bounds->keep[1][first + t]) << 1;
    const unsigned long long mask = __ballot(f != 0);
    int at = 0;
    if (x.lane == 0 && mask) at = atomicAdd(&x.bounds->left, __popcll(mask));
    at = __builtin_amdgcn_readfirstlane(at) + __popcll(mask & ((1ull << x.lane) - 1ull));
    if (f) x.bounds->index[at] = uint16_t(first + t + (f << 8));
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(x.bounds->left);
}

// Evaluates a list for the 4 x 4 cells of every wave.  The four waves fetch the 16 operand rows of a split, 16 bytes a
// lane, two batches ahead, and pass them through LDS.  `between` runs behind the first requests.
template <bool BOUNDS, class F>
__device__ __forceinline__ void flow_splits(Flow<BOUNDS>& x, int first, int n, double (&key)[4][4], int& half, bool low, F&& between) {
    auto& s = x.s;
    const int L = x.L, lane = x.lane, wq = x.wq, h = 4 * (wq & 1), lr = lane >> 4, lc = 4 * (lane & 15);
    // what this wave fetches: waves 0, 1 the left rows, waves 2, 3 the right ones
    const bool right = wq >= 2;
    const uint32_t step = uint32_t(right ? h + lr : row_base(L, x.i0 + h + lr) - row_base(L, x.i0)) * x.rowpitch;
    const int col4 = right && h + lr >= x.cend ? -kFar : 4 * (x.m0 + lc);
    u32x4 st[2][kBatch];
    const int2* list = &s.split[right ? 1 : 0][BOUNDS ? 0 : first];
    auto entry = [&](int k) { return BOUNDS ? int(x.bounds->index[k] & 255u) : k; };
    auto request = [&](u32x4 (&w)[kBatch], int k) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int2 e = list[entry(k + u)];
            const int col = col4 - e.y;
            const uint32_t at = step + uint32_t(e.x) + uint32_t(max(col, 0));
            w[u] = tld4_dev(x.tab, at | (col > -16 ? 0u : kNoRead));
        }
    };
    auto deposit = [&](const u32x4 (&w)[kBatch], int k) {
        u32x4* to = reinterpret_cast<u32x4*>(&s.u.buf[half][0][wq * 4 + lr][lc]);
        constexpr int next = 2 * kT * 64 / 4;
        if (low && right) {  // uniform: a shift may end inside a lane's four columns
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int d = list[entry(k + u)].y - col4;
                const u32x4 a = w[u];
                // columns below zero are infeasible: minima of the first columns of sub-chunks bound others
                to[u * next] = u32x4{d > 0 ? kInf : a.x, d > 4 ? kInf : d == 4 ? a.x : a.y,
                                     d > 8 ? kInf : d == 8 ? a.x : d == 4 ? a.y : a.z, d > 12 ? kInf : d == 12 ? a.x : d == 8 ? a.y : d == 4 ? a.z : a.w};
            }
        } else {
#pragma unroll
            for (int u = 0; u < kBatch; ++u) to[u * next] = w[u];
        }
    };
    const int rq = (wq >> 1) * 4, cq = (wq & 1) * 4;
    auto evaluate = [&](int k) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (k + u >= n) break;
            if (BOUNDS && !(__builtin_amdgcn_readfirstlane(int(x.bounds->index[k + u])) >> 8 & (rq ? 2 : 1))) continue;
            const double add = s.key[BOUNDS ? entry(k + u) : first + k + u];
            double l[4], r[4];
#pragma unroll
            for (int v = 0; v < 4; ++v)
                l[v] = double(s.u.buf[half][u][rq + v][lane]), r[v] = double(s.u.buf[half][u][kT + cq + v][lane]) + add;
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int d = 0; d < 4; ++d) key[a][d] = fmin(key[a][d], l[a] + r[d]);
        }
    };
    if (n) request(st[0], 0), request(st[1], kBatch);
    between();
    auto turn = [&] {  // one buffer: until it has been read; two: the other one has
        if constexpr (BOUNDS) __syncthreads();
        else half ^= 1;
    };
    for (int k = 0; k < n; k += 2 * kBatch) {
        deposit(st[0], k);
        __syncthreads();
        if (k + 2 * kBatch < n) request(st[0], k + 2 * kBatch);
        evaluate(k);
        turn();
        if (k + kBatch >= n) break;
        deposit(st[1], k + kBatch);
        __syncthreads();
        if (k + 3 * kBatch < n) request(st[1], k + 3 * kBatch);
        evaluate(k + kBatch);
        turn();
    }
}

// Without bounds 131 registers and 46 KB of LDS, three work-groups a compute unit; with them 128 and 38 KB, four (one buffer for operands instead of two;
// with three 1 x 192 stages, 4096 slots took 727 us instead of 666).  The frontier (ws.need) must not change while the kernel runs: what a
// work-group does by it is decided by several waves.
template <bool BOUNDS>
__global__ void __launch_bounds__(kFlow, BOUNDS ? 4 : 3) flow_kernel(Ctx c, int B) {
    constexpr int T = kT, NBUF = FlowLds<BOUNDS>::NBUF;
    __shared__ FlowLds<BOUNDS> s;
    __shared__ std::conditional_t<BOUNDS, FlowBounds, int> sb;
    const int L = c.L, pitch = c.pitch, nblk = blocks_of(L), chunks = pitch / 64, lane = threadIdx.x & 63;
    const int b = int(blockIdx.x) % B;
    const int words = prog_words(pitch);
    int32_t* prog = c.ws.prog + size_t(b) * tiles_of(L) * words;
    if (threadIdx.x == 0) {
        s.ticket = atomicAdd(prog + chunks, 1);  // the chain's counter stands with its first tile
        s.fault = __hip_atomic_load(c.ws.fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        s.reach = prog[(tiles_of(L) - 1) * words + chunks];
        s.n_edge = s.n_inner = 0;
    }
    if constexpr (!BOUNDS) s.split[0][threadIdx.x] = s.split[1][threadIdx.x] = make_int2(0, kFar);  // reads nothing
    __syncthreads();
    const FlowPlace at = flow_place(__builtin_amdgcn_readfirstlane(s.ticket), nblk, chunks, lane);
    if (at.D >= nblk || at.band < 0) return;  // cannot happen: one ticket per work-group
    const int D = at.D, band = at.band, I = at.I, J = I + D;
    const size_t chain = size_t(b) * c.rows * pitch;
    const size_t bl = size_t(b) * L;
    FlowBounds* bounds = nullptr;
    if constexpr (BOUNDS) bounds = &sb;
    Flow<BOUNDS> x{c, s, bounds, table_rsrc(c.cost + chain, uint32_t(c.rows) * uint32_t(pitch) * 4u),
           __builtin_amdgcn_make_buffer_rsrc(c.arg + chain, 0, int(uint32_t(c.rows) * uint32_t(pitch)), 0x00020000), prog,
           b, I, J, D, L, pitch, I * T, J * T, min(T, L - J * T), band * 64, lane,
           __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6)), uint32_t(pitch) * 4u, bl};
    if (s.fault != 0) return;  // an earlier work-group gave up: drain
    const uint32_t rp = x.rowpitch;
    const int wq = x.wq, i0 = x.i0, j0 = x.j0, cend = x.cend, m0 = x.m0;
    {   // parameters of the tile
        const int t = threadIdx.x;
        const int32_t* P = c.ws.P + size_t(b) * (L + 1);
        if (t < 64) {
            const int r = t >> 3, cc = t & 7;
            const size_t at = (bl + min(i0 + r, L - 1)) * L + min(j0 + cc, L - 1);
            reinterpret_cast<int2*>(&s.gate[r][cc & 3])[cc >> 2] = make_int2(c.ws.mall[at], c.ws.mnull[at]);
            int need = cc >= (D == 0 ? r : 0) && cc < cend && i0 + r < L ? c.ws.need[at] : 1 << 30;
#pragma unroll
            for (int o = 4; o > 0; o >>= 1) need = min(need, __shfl_xor(need, o));
            if (cc == 0) s.rows[r].need = need;
        } else if (t < 128) {
            const int e = t - 64;
            if (D == 0) {
            } else if (e < kLeft) {  // left operand (i0 + r, i0 + v)
                const int r = (e >= 8) + (e >= 15) + (e >= 21) + (e >= 26) + (e >= 30) + (e >= 33) + (e >= 35), v = e - (r * T - r * (r - 1) / 2) + r;
                s.item[e] = make_int4(int(uint32_t(tri_row(L, i0 + r, i0 + v)) * rp), 0, 16 * v & 63, 0);
            } else {  // right operand (q, j0 + cc) of split q = j0 + c2 + 1
                const int p = e - kLeft, c2 = (p >= 7) + (p >= 13) + (p >= 18) + (p >= 22) + (p >= 25) + (p >= 27);
                const int cc = p - c2 * (2 * T - 1 - c2) / 2 + c2 + 1, q = min(j0 + c2 + 1, L - 1);
                s.item[e] = make_int4(int(cc < cend ? uint32_t(row_base(L, q) + j0 + cc) * rp : kNoRead), c.ws.wsh[bl + q], 16 * cc & 63, 0);
            }
        } else if (t < 128 + T) {
            const int r = t - 128, i = min(i0 + r, L - 1), u = min(i0 + r + 1, L - 1);
            FlowRow& w = s.rows[r];
            w.sh = 4 * c.ws.wsh[bl + u], w.wab = 4 * c.ws.wabs[bl + i];
            w.Pu = P[u], w.fb = c.ws.fb[bl + i], w.P = P[i];
            w.under = int(uint32_t(row_base(L, u) + j0) * rp), w.own = int(uint32_t(row_base(L, i) + j0) * rp);
        } else if (t >= 192 && t < 192 + T) {
            s.Pj[t - 192] = P[min(j0 + t - 192 + 1, L - 1)];
        }
    }
    // the splits whose operands the neighbours finish, and those whose operands are older
    const int ne = D == 0 ? 0 : D == 1 ? 1 : D == 2 ? 9 : 16, ni = D > 2 ? 8 * (D - 3) + 1 : 0, inner = i0 + 2 * T;
    if constexpr (BOUNDS) {  // an entry a thread
        const int k = threadIdx.x;
        if (k < kEdge ? k < ne : k - kEdge < ni) {
            const int q = k >= kEdge ? inner + k - kEdge : D > 2 && k >= 8 ? j0 - T + k - 7 : i0 + T + k;
            const int sh = c.ws.wsh[bl + q], Pq = c.ws.P[size_t(b) * (L + 1) + q];
            s.split[0][k] = make_int2(int(uint32_t(row_base(L, i0) + q - 1) * rp), 0);
            s.split[1][k] = make_int2(int(uint32_t(row_base(L, q) + j0) * rp), 4 * sh);
            s.key[k] = double(Pq) + double(q + 1) * (1.0 / 256.0) + kKeyBase;
            sb.qp[k] = make_int2(q, Pq);
        } else {
            s.split[0][k] = s.split[1][k] = make_int2(0, kFar);  // reads nothing
        }
    }
    if (J + 1 < nblk) mark_tile(x, J + 1);
    __syncthreads();
    int tile_need = 1 << 30;
#pragma unroll
    for (int r = 0; r < T; ++r) tile_need = min(tile_need, s.rows[r].need);
    const bool empty = m0 + 63 < tile_need;  // below the frontier of every cell
    auto ready = [&](int back, int below) {  // the neighbours back diagonals down, this band and `below` chunks under it
        if (wq == 0 && !wait_tiles(x, tile_index(nblk, I, J - back), tile_index(nblk, I + back, J), band, below)) {
            if (lane == 0) {
                __hip_atomic_store(c.ws.fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                s.fault = 1;
            }
        }
        __syncthreads();
        return s.fault == 0;
    };
    const int operands = ckpt_rules::operand_chunks(s.reach), samples = ckpt_rules::sample_chunks(s.reach);
    uint32_t leftL[T], leftH[T], colL[T], colH[T], alL = 0, alH = 0;
#pragma unroll
    for (int r = 0; r < T; ++r) leftL[r] = leftH[r] = colL[r] = colH[r] = 0;
    int evaluated = 0;
    if (empty) {
        // the neighbours first: one of them marks these cells, and whoever sees this tile finished relies on both
        if (D > 0 && !ready(1, operands)) return;
        for (int k = wq; k < 2 * T; k += 4) {
            const int e = k * 4 + (lane >> 4), r = e >> 3, cc = e & 7;
            const bool is = i0 + r < L && cc < cend && (D != 0 || cc >= r);
            const uint32_t at = uint32_t(tri_row(L, i0 + r, j0 + cc)) * uint32_t(pitch) + uint32_t(m0 + 4 * (lane & 15));
            tst4<16>(x.tab, int(is ? at * 4u : kNoRead), u32x4{kInf, kInf, kInf, kInf});
            __builtin_amdgcn_raw_buffer_store_b32(0, x.atab, int(is ? at : kNoRead), 0, 0);
        }
        if (BOUNDS) {
            const int r = int(threadIdx.x) >> 5, kk = (threadIdx.x >> 3) & 3;
            const uint32_t line = uint32_t(pitch / kG) * uint32_t(4 * T);
            const rsrc_t smp = table_rsrc(c.ws.samp + size_t(b) * samp_ints(L, pitch), uint32_t(samp_rows(L)) * line);
            const uint32_t at = uint32_t(4 * J * (J + 1) + i0 + r) * line + (uint32_t(m0 / kG + kk) * T + (threadIdx.x & 7)) * 4u;
            __builtin_amdgcn_raw_buffer_store_b32(int(kInf), smp, int(i0 + r < L ? at : kNoRead), 0, 16);
        }
    } else if (D > 0) {
        double key[4][4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) key[r][cc] = kKeyBase + 4294967295.0;
        int half = 0;
        const bool low = s.reach > m0;
        if constexpr (!BOUNDS) {  // the first wave looks at the neighbours meanwhile
            if (wq == 1) {
                const int k = min(lane, ne - 1);
                list_splits(x, D > 2 && k >= 8 ? j0 - T + k - 7 : i0 + T + k, lane < ne, 0, &s.n_edge);
            } else if (wq > 1) {
                for (int k = 64 * (wq - 2); k < ni; k += 128) list_splits(x, inner + min(k + lane, ni - 1), k + lane < ni, kEdge, &s.n_inner);
            }
        }
        const rsrc_t smp = table_rsrc(c.ws.samp + (BOUNDS ? size_t(b) * samp_ints(L, pitch) : 0), BOUNDS ? uint32_t(samp_rows(L)) * uint32_t(pitch / kG) * uint32_t(4 * T) : 0);
        if constexpr (BOUNDS) {
            const int t = threadIdx.x;
            (&sb.ub[0][0][0])[t] = kInf - 1 + uint32_t(s.rows[(t >> 7) * 4 + ((t & 31) >> 3)].P);
            sb.index[t] = kFlow - 1;  // an entry that reads nothing
            if (t == 0) sb.left = 0;
        }
        if (D > 2) {
            if (!ready(2, BOUNDS ? samples : operands)) return;
            int n = BOUNDS ? ni : __builtin_amdgcn_readfirstlane(s.n_inner);
            if constexpr (BOUNDS) {
                if (n > 16) {
                    lower_bounds<2>(x, smp, kEdge, n, [&] {
                        upper_bounds(x, smp, kEdge, n);
                        __syncthreads();
                    });
                    __syncthreads();
                }
                n = left_over(x, kEdge, n, n <= 16);
            }
            flow_splits<BOUNDS>(x, kEdge, n, key, half, low, [] {});
            evaluated = n;
            if constexpr (BOUNDS) {
                // what is evaluated bounds the cells from above: a minimum at the first column of a sub-chunk
                if ((lane & 15) == 0) {
#pragma unroll
                    for (int a = 0; a < 4; ++a)
#pragma unroll
                        for (int d = 0; d < 4; ++d)
                            atomicMin(&sb.ub[wq >> 1][lane >> 4][a * T + (wq & 1) * 4 + d], uint32_t(__builtin_bit_cast(unsigned long long, key[a][d]) >> 8));
                }
                __syncthreads();  // the list has been read
                sb.index[threadIdx.x] = kFlow - 1;
                if (threadIdx.x == 0) sb.left = 0;
            }
        }
        // The operands of the rows from the tiles (I, I) and (J, J).  Whatever is finished two diagonals down has waited for these, so
        // they can be here before the last neighbours have finished: us a solve so and behind those, 5 x 53 stages, 777 slots
        // 105 and 109;  10 x 50, 500 slots 94 and 99;  2 x 61, 3002 slots 168 and 173.  With bounds there are no registers to hold them meanwhile.
        const int k4 = lane & 3, cb = wq * 16 + (lane >> 2), mine = (cb + 16 * k4) & 63, lr = lane >> 4, lc = 4 * (lane & 15);
        u32x4 st[4];
        auto request_rows = [&] {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int4 it = s.item[(4 * wq + k) * 4 + lr];
                const int col = m0 + lc - it.y;
                st[k] = tld4_dev(x.tab, uint32_t(it.x) != kNoRead && col > -4 ? uint32_t(it.x) + 4u * uint32_t(max(col, 0)) : kNoRead);
            }
        };
        auto settle_rows = [&] {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int4 it = s.item[(4 * wq + k) * 4 + lr];
                if (low) {  // a shift may end inside a lane's four columns
                    const u32x4 v = st[k];
                    const int d = it.y - m0 - lc;
                    if (d == 1) st[k] = u32x4{0, v.x, v.y, v.z};
                    if (d == 2) st[k] = u32x4{0, 0, v.x, v.y};
                    if (d == 3) st[k] = u32x4{0, 0, 0, v.x};
                }
                *reinterpret_cast<u32x4*>(&s.u.stage[NBUF - 1][(4 * wq + k) * 4 + lr][(lc + it.z) & 63]) = st[k];
            }
            __syncthreads();
#pragma unroll
            for (int r = 0; r < T; ++r) {
                const int at = r * T - r * (r - 1) / 2 - r;  // + column
                if (r < 4) leftL[r] = s.u.stage[NBUF - 1][at + max(k4, r)][r == 0 ? mine : (cb + 16 * max(k4, r)) & 63];
                leftH[r] = s.u.stage[NBUF - 1][at + max(k4 + 4, r)][r <= 4 ? mine : (cb + 16 * max(k4 + 4, r)) & 63];
            }
#pragma unroll
            for (int c2 = 0; c2 < T - 1; ++c2) {
                const int at = kLeft + c2 * (2 * T - 1 - c2) / 2 - c2 - 1;
                if (c2 < 3) {
                    const int cc = max(k4, c2 + 1);
                    const uint32_t v = s.u.stage[NBUF - 1][at + cc][(cb + 16 * cc) & 63];
                    colL[c2] = k4 > c2 ? v + uint32_t(s.Pj[c2]) : kHuge;
                }
                const int cc = max(k4 + 4, c2 + 1);
                const uint32_t v = s.u.stage[NBUF - 1][at + cc][(cb + 16 * cc) & 63];
                colH[c2] = k4 + 4 > c2 ? v + uint32_t(s.Pj[c2]) : kHuge;
            }
            __syncthreads();  // the staged rows have been read
        };
        const bool early = !BOUNDS && D > 1;
        if (early) {
            if (D == 2) {
                if (!ready(2, operands)) return;
            } else {
                __syncthreads();  // the last splits have been read
            }
            request_rows();
            settle_rows();
        }
        if (!ready(1, operands)) return;
        if (!early) request_rows();
        {   // row 7's operands of C_all
            const int m = m0 + cb;
            const FlowRow w = s.rows[T - 1];
            const uint32_t o = uint32_t(k4) * rp + uint32_t(4 * m) - uint32_t(w.wab) + uint32_t(w.under);
            alL = tld_dev(x.tab, 4 * m >= w.wab && k4 < cend ? o : kNoRead, 0);
            alH = tld_dev(x.tab, 4 * m >= w.wab && k4 + 4 < cend ? o + 4 * rp : kNoRead, 0);
        }
        half = 0;
        int n = BOUNDS ? ne : __builtin_amdgcn_readfirstlane(s.n_edge);
        if constexpr (BOUNDS) {
            if (D > 2) {
                lower_bounds<1>(x, smp, 0, n, [] {});
                __syncthreads();
            }
            n = left_over(x, 0, n, D <= 2);
        }
        evaluated += n;
        flow_splits<BOUNDS>(x, 0, n, key, half, low, [&] {
            if (!early) settle_rows();
        });
        __syncthreads();
        const int rq = (wq >> 1) * 4, cq = (wq & 1) * 4;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                const unsigned long long bits = __builtin_bit_cast(unsigned long long, key[a][d]);
                const int at = (lane + 16 * (cq + d)) & 63;
                s.u.p.part[(rq + a) * T + cq + d][at] = uint32_t(bits >> 8);
                s.u.p.pnum[(rq + a) * T + cq + d][at] = uint8_t(bits);
            }
        __syncthreads();
        flow_rows<false, BOUNDS>(x, leftL, leftH, colL, colH, alL, alH);
    } else {
        flow_rows<true, BOUNDS>(x, leftL, leftH, colL, colH, 0, 0);
    }
    // operands of the evaluated splits; 64 rows for the splits of the row and column blocks, eight for C_all of row 7
    if (c.work && wq == 0)
        count_work<true>(c.work, 2, unsigned(empty || D == 0 ? 0 : 16 * evaluated + 72), unsigned(D == 0 ? cend * (cend + 1) / 2 : T * cend));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);  // the stores are through
    __syncthreads();
    if (threadIdx.x == 0) __hip_atomic_store(prog + size_t(tile_index(nblk, I, J)) * words + band, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// ---------------------------------------------------------------------------
// Short chains (chain_kernel): one launch, a work-group per chain, thread = column.  The cells of the whole table but its first
// row (nobody reads that) stand in LDS, so nothing waits for memory but the first reads of the chain, and the thresholds are
// computed by the first wave: no table of them, no marks, no tickets.  Rows bottom-up with a barrier each; left operands are
// the thread's own cells of the row, right operands and those of C_all come from LDS at a shifted column.  A column
// below zero reads column 0: its gate is closed.  The barriers wait for LDS and not for the stores.  Rows, cells and splits are
// unrolled (with a loop over the rows, which needs a test a split, 1 x 8 stages, 64 slots take 11.1 us instead of 7.2), and what
// belongs to a split is held by every thread (in scalar registers it spilled: 200 x 13, 500 slots 32 us instead of 24).
// What bounds it: up to eight stages the launch and the first reads; longer chains the few waves that a chain's columns fill, with
// 6 vector instructions a split and 20 a cell.  200 x 13 stages, 500 slots: a wave issues 3500 of them in 48700 clocks, two waves a SIMD, and
// waits for LDS, the barriers and its stores 48 % of the time.  1 x 8 stages, 64 slots 10.0 -> 7.2 us a solve, 200 x 13, 500 slots 49 -> 23
// (the rule: ckpt_rules::chain_pays).
// ---------------------------------------------------------------------------
template <int N>
__global__ void __launch_bounds__(1024) chain_kernel(ckpt_chains_t ch, int L, int pitch, Workspace ws, int32_t* __restrict__ cost,
                                                      uint8_t* __restrict__ arg, unsigned long long* work) {
    extern __shared__ uint32_t s_cell[];  // rows 1 .. L - 1
    __shared__ int s_a[N + 1], s_d[N + 1], s_ab[N], s_of[N], s_ob[N];
    __shared__ int s_P[N + 1], s_sh[N], s_wabs[N], s_fb[N];
    __shared__ int2 s_gate[N][N];  // m_all, m_null
    const int b = blockIdx.x, tid = threadIdx.x;
    if (tid < 64) {
        const bool tensor = tid <= L, stage = tid < L;
        const size_t at = size_t(b) * L + tid;
        const int a_in = tensor ? ch.wa[at + b] : 0, d_in = tensor ? (ch.wdelta ? ch.wdelta : ch.wa)[at + b] : 0;
        const int ab_in = stage ? ch.wabar[at] : 0, f = stage ? ch.uf[at] : 0, bw = stage ? ch.ub[at] : 0;
        const int of_in = stage && ch.of ? ch.of[at] : 0, ob_in = stage && ch.ob ? ch.ob[at] : 0;
        const int a_next = __shfl_down(a_in, 1);
        auto sz = [](int v) { return min(max(v, 0), 1 << 28); };  // as in precompute_kernel
        const int fc = min(max(f, 0), (1 << 30) - 1), bc = min(max(bw, 0), 1 << 30);
        if (tensor) s_a[tid] = sz(a_in), s_d[tid] = sz(d_in);
        if (stage) {
            s_ab[tid] = sz(ab_in), s_of[tid] = sz(of_in), s_ob[tid] = sz(ob_in);
            s_sh[tid] = min(max(a_in, 0), pitch), s_wabs[tid] = min(max(ab_in, 0), pitch);
            s_fb[tid] = int(min(kInf, uint32_t(fc) + uint32_t(bc)));
        }
        const int sum = wave_scan(fc, [](int x, int y) { return int(min(uint32_t(x) + uint32_t(y), kInf)); });
        if (tid == 0) s_P[0] = 0;
        if (stage) s_P[tid + 1] = min(sum, int(kInf) - 1);
        int flags = 0;
        if (f < 0 || bw < 0) flags |= 1;
        if (f >= (1 << 30) || bw >= (1 << 30) || sum >= int(kInf)) flags |= 2;
        for (int v : {a_in, d_in, ab_in, of_in, ob_in}) {
            if (v < 0) flags |= 1;
            if (v > (1 << 28)) flags |= 4;
        }
        if (stage && ab_in < a_next) flags |= 8;
        flags = wave_scan(flags, [](int x, int y) { return x | y; });
        if (tid == 63) {
            ws.flags[b] = flags;
            if (b == 0) ws.fault[0] = 0;
        }
        wave_settle();
        for (int e = tid; e < N * N; e += 64) {
            const int r = e / N, t = e % N + 1;  // stages r + 1 to t, counted from one
            if (r >= t || t > L) continue;
            int most = s_a[r + 1] + s_of[r];
            for (int j = r + 2; j < t; ++j) most = max(most, s_a[j - 1] + s_a[j] + s_of[j - 1]);
            s_gate[r][t - 1] = make_int2(max(s_d[t] + s_of[r], s_d[r + 1] + s_ob[r]) + s_ab[r], s_d[t] + most);
        }
    }
    __syncthreads();
    const int row4 = pitch * 4;
    const char* cells = reinterpret_cast<const char*>(s_cell);
    const int m = tid, m4 = 4 * tid;
    // The column of cell (q, q) that a shift of `shift` slots leads to; cell (q, j) is j - q rows further.
    auto column = [&](int q, int shift) { return cells + ckpt_rules::chain_row(L, min(q, L)) * row4 + max(m4 - 4 * shift, 0); };
    auto cell = [&](const char* at, int down) { return *reinterpret_cast<const uint32_t*>(at + down * row4); };
    const char* from[N];  // of split q
    uint32_t P[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
        const int u = min(q, L - 1);
        from[q] = column(max(q, 1), s_sh[u]), P[q] = uint32_t(s_P[u]);
    }
    int32_t* ctab = cost + size_t(b) * (size_t(L) * (L + 1) / 2) * pitch;
    uint8_t* atab = arg + size_t(b) * (size_t(L) * (L + 1) / 2) * pitch;
    unrolled<N>([&](auto step) {
        constexpr int i = N - 1 - decltype(step)::value;
        if (i >= L) return;  // uniform
        {
            uint32_t val[N];
            const char* under = column(i + 1, s_wabs[i]);
            const uint32_t fb = uint32_t(s_fb[i]);
#pragma unroll
            for (int j = i; j < N; ++j) {
                if (j >= L) break;  // uniform
                const int2 gate = s_gate[i][j];
                uint32_t best = kInf, pick = 0;
#pragma unroll
                for (int q = i + 1; q <= j; ++q) {
                    const uint32_t v = val[q - 1] + (P[q] - P[i]) + cell(from[q], j - q);
                    pick = q == i + 1 || v < best ? uint32_t(q + 1) : pick;
                    best = q == i + 1 ? v : min(v, best);
                }
                uint32_t all = fb;
                if (j > i) all += cell(under, j - i - 1);
                const uint32_t ck = m >= gate.y ? best : kInf;
                all = m >= gate.x ? all : kInf;
                pick = all <= ck ? uint32_t(i + 1) : pick;
                val[j] = min(min(all, ck), kInf);
                pick = val[j] < kInf ? pick : 0u;
                const size_t at = size_t(tri_row(L, i, j)) * pitch + m;
                if (i > 0) s_cell[at - size_t(L) * pitch] = val[j];
                ctab[at] = int32_t(val[j]);
                atab[at] = uint8_t(pick);
            }
            if (work) count_work<true>(work, 2, 0, unsigned(L - i));
        }
        if (i > 0) {  // for LDS: the stores to memory are nobody's business
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        }
    });
}

using RowFn = void (*)(Ctx, int);
template <int T, int DC, int... Rs>
constexpr std::array<RowFn, sizeof...(Rs)> row_table(std::integer_sequence<int, Rs...>) {
    return {{row_kernel<T, Rs, DC>...}};
}
const std::array<RowFn, kT> kRow0 = row_table<kT, 0>(std::make_integer_sequence<int, kT>{});
const std::array<RowFn, kT> kRow1 = row_table<kT, 1>(std::make_integer_sequence<int, kT>{});
const std::array<RowFn, kT> kRow2 = row_table<kT, 2>(std::make_integer_sequence<int, kT>{});


// ---------------------------------------------------------------------------
// Planner-side steps (Section "Integrate Two Solvers").
// ---------------------------------------------------------------------------

// One block: lexicographic minimum of (C_BP(1, L, m_b), b) over the chains.
__global__ void __launch_bounds__(256) select_kernel(const int32_t* __restrict__ cost, int L, int M, int pitch,
                                                      int rows, int B, const int32_t* __restrict__ m_budget,
                                                      int32_t* __restrict__ out) {
    __shared__ unsigned long long s_best[256];
    const size_t root = size_t(tri_row(L, 0, L - 1)) * pitch;
    unsigned long long best = (static_cast<unsigned long long>(kInf) << 32) | 0xffffffffull;
    for (int b = threadIdx.x; b < B; b += blockDim.x) {
        const int m = m_budget[b];
        if (m < 0) continue;
        const uint32_t v = uint32_t(cost[size_t(b) * rows * pitch + root + min(m, M)]);
        if (v < kInf) best = min(best, (static_cast<unsigned long long>(v) << 32) | uint32_t(b));
    }
    s_best[threadIdx.x] = best;
    __syncthreads();
    for (int o = blockDim.x / 2; o > 0; o >>= 1) {
        if (int(threadIdx.x) < o) s_best[threadIdx.x] = min(s_best[threadIdx.x], s_best[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const unsigned long long r = s_best[0];
        out[0] = (r >> 32) < kInf ? int32_t(r & 0xffffffffull) : -1;
        out[1] = int32_t(r >> 32);
    }
}

// slots = min(2^31 - 1, ceil(bytes * M / budget))
__device__ inline int32_t slots_of(long long bytes, unsigned long long budget, int M) {
    const unsigned long long v = static_cast<unsigned long long>(bytes) * uint32_t(M);
    const unsigned long long q = budget ? v / budget + (v % budget != 0) : 0x7fffffffull;
    return int32_t(min(q, 0x7fffffffull));
}

// One thread per element, one chain per blockIdx.y.
__global__ void __launch_bounds__(256) discretize_kernel(const long long* __restrict__ in, int32_t* __restrict__ out,
                                                          const long long* __restrict__ budget, int per_chain, int M) {
    const int b = blockIdx.y;
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= per_chain) return;
    out[size_t(b) * per_chain + k] =
        slots_of(in[size_t(b) * per_chain + k], static_cast<unsigned long long>(budget[b]), M);
}

// The same for one profile under every budget of a sweep: chain blockIdx.y uses budget[blockIdx.y], and blockIdx.x says which array is
// cut; behind the arrays, the budgets themselves.  All in one launch: what bounds it are launches, 2 us each (10 chains of
// 50 stages, a whole plan 124 -> 119 us).
struct SweepBudgets { long long v[CKPT_MAX_SWEEP]; };
struct SweepArray { const int64_t* in; int32_t* out; int n; };
struct SweepArrays { SweepArray v[5]; };
constexpr int kSweepThreads = 256;
static_assert(CKPT_MAX_L < kSweepThreads && CKPT_MAX_SWEEP <= kSweepThreads, "a thread per element");
__global__ void __launch_bounds__(kSweepThreads) discretize_sweep_kernel(SweepArrays arrays, int n_arrays, SweepBudgets budget, int count,
                                                                          long long* __restrict__ budgets_out, int M) {
    const int b = blockIdx.y, k = threadIdx.x;
    if (int(blockIdx.x) == n_arrays) {
        if (b == 0 && k < count) budgets_out[k] = budget.v[k];
        return;
    }
    const SweepArray& a = arrays.v[blockIdx.x];
    if (k < a.n) a.out[size_t(b) * a.n + k] = slots_of(a.in[k], static_cast<unsigned long long>(budget.v[b]), M);
}

// One work-group per chain walks its recorded candidates.  A walk is a tree of cells whose candidate
// numbers come from memory one dependent read after another; what bounds it is the number of such
// round trips, so the tree is taken breadth first, all pending cells at once (wave 0), and runs of C_all
// are followed ahead of their numbers: the lanes of a cell read (s + u, t, m - sum of abar^s .. abar^{s+u-1})
// together, and the first number that is not C_all ends the run.  Few pending cells get many lanes each.
// A wave by itself issues an instruction every 4 (vector) or 8 (scalar) clocks and waits 130 for each
// access to LDS, so a round is kept short: a node is one 16-byte word, what a stage adds to an address and
// to m is a second one, the ends of all runs come from one addition to the mask of the lanes that go on,
// and the read is not behind a branch.
// Positions need no pass over the tree: the operations before a cell are those that its ancestors put
// before their children and all that start right of it, and its own subtree is what starts in its stages,
// less the ancestors that start where it does.  So sums by stage place every node, and all waves write the list.
// 8 chains of 192 stages, 4096 slots (29 to 38 rounds): 26 us a call; 50 with 300 instructions a round and
// the sizes of subtrees summed round by round (10 us of it), 290 for one thread per chain with its stack
// in memory (a cell every microsecond); 10 chains of 50 stages (7 to 12 rounds): 12, 20 and 89 us.  Reading both children
// of every split a cell could have ahead of its number saves a quarter of the rounds (runs and
// right children alternate, and a run's length is not known), and three reads a stage cost more: 52 us.
// Cells below a run cover disjoint stages, so a walk has at most L leaves, L - 1 splits and L - 1 cells
// that only continue a run.
constexpr int kWalkNodes = 3 * CKPT_MAX_L;
constexpr int kWalkThreads = 256;
static_assert(CKPT_MAX_L < kWalkThreads, "tables by stage; s_total is indexed by a stage and the one after it");

__global__ void __launch_bounds__(kWalkThreads) schedule_kernel(const uint8_t* __restrict__ arg,
                                                                 const int32_t* __restrict__ wa,
                                                                 const int32_t* __restrict__ wabar, int L, int M, int pitch,
                                                                 int rows, const int32_t* __restrict__ m_budget,
                                                                 ckpt_op_t* __restrict__ ops, int cap,
                                                                 int32_t* __restrict__ n_ops) {
    enum { kLeaf = 0, kSplit = 1, kMore = 2, kBad = 3 };  // how a node ends after its run of C_all
    // A node, as one 16-byte word:
    //   x  slots of the cell, held in 32 bits (outside 0 .. M there is no cell: the node is bad)
    //   y  s | t << 8 | operations of its ancestors that come before their children's << 16 (at most L(L+1)/2 + L)
    //   z  operations of its ancestors that start at the same stage
    //   w  run | end << 8 | k << 16
    __shared__ int4 s_node[kWalkNodes + 64];  // a round's lanes look at 64 of them: those beyond the last one have s > t
    struct alignas(16) Stage {
        long long sum;  // of abar before the stage
        int row;        // offset of its cells' row in the table, less that of t = 0
        int wab;
    };
    __shared__ Stage s_stage[kWalkThreads];
    __shared__ int32_t s_wa[CKPT_MAX_L + 1];
    __shared__ int s_total[kWalkThreads + 1];  // operations of the nodes that start at a stage, then before it
    __shared__ long long s_part[kWalkThreads / 64];
    __shared__ int s_wave[kWalkThreads / 64];
    __shared__ int s_count, s_first_bad;
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint8_t* tab = arg + size_t(b) * rows * pitch;
    // Sizes of a chain that ckpt_check_inputs would flag are taken as they come: a negative one raises m.
    auto left = [](long long m, int size) { return __builtin_elementwise_sub_sat(int(m), size); };  // m in 0 .. M
    const int wab = tid > 0 && tid <= L ? wabar[size_t(b) * L + tid - 1] : 0;
    for (int k = tid; k <= L; k += kWalkThreads) s_wa[k] = wa[size_t(b) * (L + 1) + k];
    const int m0 = m_budget[b];
    if (m0 < 0) {  // uniform
        if (tid == 0) n_ops[b] = CKPT_E_ARG;
        return;
    }
    for (int i = tid; i < kWalkNodes + 64; i += kWalkThreads)
        s_node[i] = i == 0 ? make_int4(min(m0, M), 1 | L << 8, 0, 0) : make_int4(0, 1, 0, 0);
    s_total[tid] = 0;
    if (tid == 0) s_first_bad = INT32_MAX;
    long long sum = wab;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const long long w = __shfl_up(sum, o);
        if (lane >= o) sum += w;
    }
    if (lane == 63) s_part[wave] = sum;
    __syncthreads();
    for (int w = 0; w < wave; ++w) sum += s_part[w];
    s_stage[tid] = Stage{sum - wab, int(unsigned((tid - 1) * L - (tid - 1) * (tid - 2) / 2 - tid) * unsigned(pitch)), wab};
    __syncthreads();

    if (tid < 64) {
        int head = 0, tail = 1;
        while (head < tail) {  // head grows in every round, tail is bounded: see kWalkNodes
            wave_settle();
            const int n = min(tail - head, 64);
            const int log_groups = n > 1 ? 32 - __builtin_clz(n - 1) : 0;
            const int width = 64 >> log_groups, group = lane >> (6 - log_groups), u = lane & (width - 1);
            const int4 nd = s_node[head + group];
            const int s0 = nd.y & 255, t = nd.y >> 8 & 255, s = s0 + u;
            const bool here = s <= t;
            const Stage at_s = s_stage[min(s, t)];
            const long long m = nd.x - (at_s.sum - s_stage[s0].sum);
            // inside the table, and ahead of its turn a lane reads no further than this cell could
            const bool read = here & (m >= 0) & (m <= min(nd.x, M));
            const int in_table = tab[read ? unsigned(at_s.row + t * pitch + int(m)) : 0u], k = read ? in_table : 0;
            const bool goes_on = k == s && s < t;  // C_all
            const unsigned long long on = __ballot(goes_on);
            // The lane that ends the run: the first that does not go on, or the last one as a C_all cell.  A bit
            // added where each group begins carries to it.
            const unsigned long long first = __ballot(here && u == 0);
            const unsigned long long carry = on & ~(first << (width - 1)), ends = (carry + first) & ~carry;
            const unsigned long long splits = ends & __ballot(k > s) & __ballot(k <= t);
            // a size below zero raised m: not read ahead of its turn
            const unsigned long long more = ends & (on | __ballot(here && m > nd.x && m <= M));
            const unsigned long long bit = 1ull << lane;
            if (ends & bit) {
                const bool split = splits & bit, next = more & bit;
                const int run = u + (goes_on ? 1 : 0);
                const int end = next ? kMore : split ? kSplit : k == s ? kLeaf : kBad;
                s_node[head + group].w = run | end << 8 | k << 16;
                if (split || next) {
                    const int at = tail + 2 * __popcll(splits & (bit - 1)) + __popcll(more & (bit - 1));
                    const int own = split ? k - s0 : run;  // before the children
                    const int a = s_wa[split ? k - 1 : 0], slots = left(m, split ? a : goes_on ? at_s.wab : 0);
                    // (k, t, m - a^{k-1}) is walked first, then (s, k - 1, m)
                    s_node[at] = make_int4(slots, (split ? k : s0 + run) | ((nd.y & ~255) + (own << 16)), 0, 0);
                    if (split)
                        s_node[at + 1] = make_int4(int(m), s | (k - 1) << 8 | ((nd.y & ~0xffff) + (own << 16)),
                                                   u == 0 ? nd.z + own : 0, 0);
                }
            }
            tail += 2 * __popcll(splits) + __popcll(more);
            head += n;
        }
        if (lane == 0) s_count = head;
    }
    __syncthreads();
    const int count = s_count;
    struct Node {
        int s, t, before, same, run, end, k;
    };
    auto node = [&](int i) {
        const int4 nd = s_node[i];
        return Node{nd.y & 255, nd.y >> 8 & 255, int(unsigned(nd.y) >> 16), nd.z, nd.w & 255, nd.w >> 8 & 255, nd.w >> 16};
    };
    // operations before the children: the run's F_all, then F_all B of a leaf or F_ck F_null .. of a split
    auto before = [](const Node& nd) { return nd.end == kSplit ? nd.k - nd.s : nd.run + (nd.end == kLeaf ? 2 : 0); };
    for (int i = tid; i < count; i += kWalkThreads) {
        const Node nd = node(i);
        atomicAdd(&s_total[nd.s], before(nd) + nd.run);
    }
    __syncthreads();
    int upto = s_total[tid];
    const int here = upto;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int w = __shfl_up(upto, o);
        if (lane >= o) upto += w;
    }
    if (lane == 63) s_wave[wave] = upto;
    __syncthreads();
    for (int w = 0; w < wave; ++w) upto += s_wave[w];
    s_total[tid] = upto - here;
    if (tid == kWalkThreads - 1) s_total[kWalkThreads] = upto;
    __syncthreads();
    const int n = s_total[kWalkThreads];
    auto position = [&](const Node& nd) { return nd.before + n - s_total[nd.t + 1]; };
    for (int i = tid; i < count; i += kWalkThreads) {
        const Node nd = node(i);
        if (nd.end == kBad) atomicMin(&s_first_bad, position(nd) + before(nd));
    }
    __syncthreads();
    const int bad = s_first_bad;
    const int limit = min(cap, bad);  // the list ends where the walk in order would have ended
    ckpt_op_t* out = ops + size_t(b) * cap;
    auto emit = [&](int at, int kind, int stage) {
        if (at < limit) out[at].kind = uint8_t(kind), out[at].stage = uint8_t(stage);
    };
    for (int i = tid >> 3; i < count; i += kWalkThreads / 8) {  // eight lanes a node
        const Node nd = node(i);
        const int s = nd.s + nd.run, x = tid & 7, first = position(nd);
        const int last = first + s_total[nd.t + 1] - s_total[nd.s] - nd.same - 1;
        for (int u = x; u < nd.run; u += 8) {
            emit(first + u, CKPT_OP_F_ALL, nd.s + u);
            emit(last - u, CKPT_OP_B, nd.s + u);
        }
        if (nd.end == kLeaf && x < 2) emit(first + nd.run + x, x ? CKPT_OP_B : CKPT_OP_F_ALL, s);
        if (nd.end == kSplit)
            for (int j = s + x; j < nd.k; j += 8) emit(first + nd.run + j - s, j == s ? CKPT_OP_F_CK : CKPT_OP_F_NULL, j);
    }
    if (tid == 0) {
        int rc = n;
        if (bad <= cap) {
            const Node nd = node(0);  // its first number is read in every case: 0 is the table's mark of an infeasible cell
            rc = nd.end == kBad && nd.run == 0 && nd.k == 0 ? CKPT_E_INFEASIBLE : CKPT_E_CORRUPT;
        } else if (n > cap || bad != INT32_MAX) {
            rc = CKPT_E_SMALLBUF;
        }
        n_ops[b] = rc;
    }
}

// Checkpoint block index of every stage (Section "Code generation"): one work-group per chain reads the
// first forward sweep of its operation list, a thread per stage.  In a list produced by the walk above, operation k
// (k < L) is the first forward of stage k + 1 and operation L is B^L; F_ck opens a block, F_null
// continues it, F_all lies in none.  The block number of a stage is the count of F_ck up to it,
// minus one: bits of a ballot.  Bounded by the launch and one read, which does not wait for the length
// of the list: 8 chains of 192 stages 3.1 us, 3.8 for one wave in passes of 64 stages.
constexpr int kBlockThreads = 256;
static_assert(CKPT_MAX_L < kBlockThreads, "a thread per stage and one for B^L");

__global__ void __launch_bounds__(kBlockThreads) block_index_kernel(const ckpt_op_t* __restrict__ ops, int cap,
                                                          const int32_t* __restrict__ n_ops, int L,
                                                          int32_t* __restrict__ block_of_stage,
                                                          int32_t* __restrict__ n_blocks) {
    constexpr int kWaves = kBlockThreads / 64;
    __shared__ unsigned long long s_opens[kWaves], s_inside[kWaves];
    const int b = blockIdx.x, k = threadIdx.x, lane = k & 63, wave = k >> 6;
    ckpt_op_t op{CKPT_OP_F_ALL, uint8_t(k + 1)};
    if (k <= L && k < cap) op = ops[size_t(b) * cap + k];
    const int n = n_ops[b];
    int32_t* out = block_of_stage + size_t(b) * L;
    if (n < 0 || n > cap || n < L + 1) {  // uniform: a failed walk keeps its code, a short list is corrupt
        if (k < L) out[k] = -1;
        if (k == 0) n_blocks[b] = n < 0 ? n : (n > cap ? CKPT_E_ARG : CKPT_E_CORRUPT);
        return;
    }
    const bool valid = k < L;
    const unsigned long long opens = __ballot(valid && op.kind == CKPT_OP_F_CK);
    const unsigned long long inside = __ballot(valid && (op.kind == CKPT_OP_F_CK || op.kind == CKPT_OP_F_NULL));
    if (lane == 0) s_opens[wave] = opens, s_inside[wave] = inside;
    __syncthreads();
    int before = 0, blocks = 0;  // blocks opened in earlier waves, and in all
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
        const int count = __popcll(s_opens[w]);
        if (w < wave) before += count;
        blocks += count;
    }
    const bool after_one = lane ? inside >> (lane - 1) & 1 : wave && s_inside[wave - 1] >> 63;
    bool bad = valid && (op.stage != k + 1 || op.kind > CKPT_OP_F_NULL || (op.kind == CKPT_OP_F_NULL && !after_one));
    if (k == L && (op.kind != CKPT_OP_B || op.stage != L)) bad = true;
    bad = __syncthreads_or(bad);
    if (valid) out[k] = !bad && inside >> lane & 1 ? before + __popcll(opens & (~0ull >> (63 - lane))) - 1 : -1;
    if (k == 0) n_blocks[b] = bad ? CKPT_E_CORRUPT : blocks;
}

// Self-check of operation lists: one work-group per chain executes its list under the memory model
// of Table 1 ("List of Operations").  What is resident of stage x (bit 0 = a^x on its own, bit 1 =
// abar^x, bit 2 = delta^x) depends only on the operations on stages x and x + 1, in their order, as long
// as none of them finds an operand missing -- and then the list is corrupt whatever follows.  So a thread
// takes a stage and steps through its own operations (found by a bit mask per stage), all stages
// at once; the thread of an operation's input stage also notes by how much the operation changes the
// resident sum.  Then a thread takes four operations: prefix sums give the memory before each one.
// What bounds it: the operations of the busiest stage, some 60 instructions each by a lone wave a SIMD.  So a
// thread goes from one of its operations to the next whatever the other lanes do, kinds are two bits that come with a
// word of its mask, empty words are not looked at, and the list is asked for before its length is known.
// 8 chains of 192 stages: 8 us; 16 with the words of the masks taken by all lanes together, 210 for one
// lane stepping through the whole list.
constexpr int kSimThreads = 256;  // at least CKPT_MAX_L + 1 stages and the empty mask after them
constexpr int kSimPer = 4;        // operations of a thread in a pass, one after another in the list
constexpr int kSimChunk = kSimPer * kSimThreads;  // operations staged per pass
static_assert(CKPT_MAX_L + 2 <= kSimThreads, "a thread per stage");
static_assert(kSimChunk == 32 * 32, "a word of s_any has a bit for every word of a mask");

__global__ void __launch_bounds__(kSimThreads) simulate_kernel(ckpt_chains_t ch, int L, const ckpt_op_t* __restrict__ ops,
                                                                int cap, const int32_t* __restrict__ n_ops,
                                                                long long* __restrict__ time_out,
                                                                long long* __restrict__ peak_out,
                                                                int32_t* __restrict__ status) {
    constexpr int kWords = kSimChunk / 32, kWaves = kSimThreads / 64;
    __shared__ int2 s_forward[CKPT_MAX_L], s_backward[CKPT_MAX_L];  // time and overhead of stage x + 1
    __shared__ int32_t s_made[2][CKPT_MAX_L];                       // a and abar of stage x + 1
    __shared__ uint32_t s_mask[kWords][kSimThreads];  // [word][stage]: which operations of the pass are the stage's
    __shared__ uint32_t s_any[kSimThreads];           // [stage]: which words of its mask are not empty
    __shared__ uint32_t s_kind[kWords][2];            // the two bits of an operation's kind
    __shared__ __align__(16) long long s_delta[kSimChunk];
    __shared__ long long s_total[kWaves], s_peak[kWaves], s_time[kWaves];
    const int b = blockIdx.x, x = threadIdx.x, lane = x & 63, wave = x >> 6;
    const ckpt_op_t* list = ops + size_t(b) * cap;
    ckpt_op_t op[kSimPer];
    auto fetch = [&](int base, int end) {
#pragma unroll
        for (int u = 0; u < kSimPer; ++u) {
            op[u] = ckpt_op_t{};
            if (base + kSimPer * x + u < end) op[u] = list[base + kSimPer * x + u];
        }
    };
    fetch(0, cap);
    const int32_t* wd = ch.wdelta ? ch.wdelta : ch.wa;
    // of stage x: a, delta; of stage x + 1: a, abar, delta
    long long a = 0, d = 0, a1 = 0, ab1 = 0, d1 = 0;
    const long long d_last = wd[size_t(b) * (L + 1) + L];
    if (x <= L) {
        a = x ? ch.wa[size_t(b) * (L + 1) + x] : 0;  // the chain input a^0 is not counted
        d = wd[size_t(b) * (L + 1) + x];
    }
    if (x < L) {
        a1 = ch.wa[size_t(b) * (L + 1) + x + 1];
        d1 = wd[size_t(b) * (L + 1) + x + 1];
        ab1 = ch.wabar[size_t(b) * L + x];
        s_forward[x] = make_int2(ch.uf[size_t(b) * L + x], ch.of ? ch.of[size_t(b) * L + x] : 0);
        s_backward[x] = make_int2(ch.ub[size_t(b) * L + x], ch.ob ? ch.ob[size_t(b) * L + x] : 0);
        s_made[0][x] = int32_t(a1), s_made[1][x] = int32_t(ab1);
    }
    const int n = n_ops[b];
    if (n < 0 || n > cap) {  // uniform over the work-group
        if (x == 0) {
            status[b] = n < 0 ? n : CKPT_E_ARG;
            time_out[b] = peak_out[b] = -1;
        }
        return;
    }
    int state = x == 0 ? 1 : x == L ? 4 : 0;  // a^0 and delta^L are there from the start
    bool bad = false;
    long long time = 0, peak = 0, carry = d_last;
    for (int base = 0; base < n; base += kSimChunk) {  // n is uniform over the work-group
        const int count = min(kSimChunk, n - base), words = (count + 31) / 32;
        for (int w = 0; w < words; ++w) s_mask[w][x] = 0;
        s_any[x] = 0;
        if (x < 2 * kWords) s_kind[x >> 1][x & 1] = 0;
        __syncthreads();
        int kind[kSimPer], stage[kSimPer];
        uint32_t bits[2] = {0, 0};
#pragma unroll
        for (int u = 0; u < kSimPer; ++u) {
            const int k = kSimPer * x + u;
            kind[u] = op[u].kind, stage[u] = op[u].stage;
            if (k >= count) continue;
            if (stage[u] < 1 || stage[u] > L || kind[u] > CKPT_OP_B) {
                bad = true;
            } else {
                atomicOr(&s_mask[k >> 5][stage[u]], 1u << (k & 31));
                atomicOr(&s_any[stage[u]], 1u << (k >> 5));
                bits[0] |= uint32_t(kind[u] & 1) << (k & 31), bits[1] |= uint32_t(kind[u] >> 1) << (k & 31);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) atomicOr(&s_kind[kSimPer * x >> 5][h], bits[h]);
        const int next_base = base + kSimChunk;
        if (next_base < n) fetch(next_base, n);  // uniform
        __syncthreads();
        if (x <= L) {
            uint32_t any = s_any[x] | s_any[x + 1], todo = 0, next = 0, kind0 = 0, kind1 = 0;
            int w = 0;
            while (any | todo) {
                if (!todo) {
                    w = __builtin_ctz(any);
                    any &= any - 1;
                    next = s_mask[w][x + 1];  // operations that read a^x: those of stage x + 1
                    todo = s_mask[w][x] | next;
                    kind0 = s_kind[w][0], kind1 = s_kind[w][1];
                }
                const int bit = __builtin_ctz(todo);
                todo &= todo - 1;
                const int what = int(kind0 >> bit & 1u) | int(kind1 >> bit & 1u) << 1;
                if (next >> bit & 1u) {  // of stage x + 1
                    const bool back = what == CKPT_OP_B, drops = what == CKPT_OP_F_NULL;
                    bad = bad || !(state & 3) || (drops && !(state & 1));
                    // B: its output is not counted while it runs; a forward operation adds its output, F_null drops its input
                    const long long gone = (back ? state & 1 : drops) ? a : 0;
                    const long long made = back ? ((state & 4) ? 0 : d) - d1 - ab1 : what == CKPT_OP_F_ALL ? ab1 : a1;
                    s_delta[32 * w + bit] = made - gone;
                    state = back ? (state & 2) | 4 : drops ? state & ~1 : state;
                } else if (what == CKPT_OP_B) {  // needs delta^x and abar^x
                    bad = bad || (state & 6) != 6;
                    state &= 1;
                } else {
                    const int made = what == CKPT_OP_F_ALL ? 2 : 1;
                    bad = bad || (state & made);
                    state |= made;
                }
            }
        }
        __syncthreads();
        long long delta[kSimPer], before = 0;
#pragma unroll
        for (int u = 0; u < kSimPer; ++u) {
            delta[u] = kSimPer * x + u < count ? s_delta[kSimPer * x + u] : 0;
            before += delta[u];
        }
        const long long own = before;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const long long v = __shfl_up(before, o);
            if (lane >= o) before += v;
        }
        if (lane == 63) s_total[wave] = before;
        __syncthreads();
        before += carry - own;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            if (w < wave) before += s_total[w];
            carry += s_total[w];
        }
#pragma unroll
        for (int u = 0; u < kSimPer; ++u) {
            const int j = min(max(stage[u], 1), L) - 1;
            const bool back = kind[u] == CKPT_OP_B, valid = kSimPer * x + u < count;
            const int2 cost = back ? s_backward[j] : s_forward[j];
            const int made = s_made[kind[u] == CKPT_OP_F_ALL][j];
            // a forward operation needs room for its output and o_f
            const long long need = before + (back ? 0 : made) + cost.y;
            if (valid) peak = max(peak, need), time += cost.x;
            before += delta[u];
        }
    }
    if (x == 0 && !(state & 4)) bad = true;  // the list must end with delta^0
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        time += __shfl_xor(time, o);
        peak = max(peak, __shfl_xor(peak, o));
    }
    if (lane == 0) s_time[wave] = time, s_peak[wave] = peak;
    bad = __syncthreads_or(bad);
    if (x == 0) {
        for (int w = 1; w < kWaves; ++w) time += s_time[w], peak = max(peak, s_peak[w]);
        status[b] = bad ? CKPT_E_CORRUPT : CKPT_OK;
        time_out[b] = bad ? -1 : time;
        peak_out[b] = bad ? -1 : peak;
    }
}

int check_dims(int L, int M, int B) {
    if (L < 1 || M < 0 || B < 1) return CKPT_E_ARG;
    if (L > CKPT_MAX_L) return CKPT_E_LIMIT;
    const unsigned long long per_chain = (unsigned long long)ckpt_table_rows(L) * ckpt_row_pitch(M);
    if (per_chain >= (1ull << 30)) return CKPT_E_LIMIT;  // 4 GiB of int32 per chain
    if (B > 65535) return CKPT_E_LIMIT;                   // chains are the z dimension of the grids
    return CKPT_OK;
}

// Optional per-launch event trail of ckpt_solve_profiled.
struct Profile {
    hipStream_t stream = nullptr;
    std::vector<hipEvent_t> events;
    std::vector<int> kinds;
    unsigned long long* work = nullptr;  // device, 4 counters
    bool trail = true;                   // record an event after every launch
    bool mark(int kind) {
        if (!trail) return true;
        hipEvent_t e;
        if (!hip_ok(hipEventCreate(&e))) return false;
        events.push_back(e);
        kinds.push_back(kind);
        return hip_ok(hipEventRecord(e, stream));
    }
};

#define CKPT_AFTER_LAUNCH(kind)                                   \
    do {                                                          \
        if (!hip_ok(hipGetLastError())) return CKPT_E_HIP;        \
        if (prof && !prof->mark(kind)) return CKPT_E_HIP;         \
    } while (0)

// Per-device state of the library, kept for the life of the process:
//   helpers  three streams (default priority, non-blocking) and five events for the batch split;
//            with the caller's stream they make four, the number of hardware queues a process
//            gets by default (more streams than that share queues and serialise: six or eight
//            groups measured slower than one).  Created by ckpt_init or by the first solve
//            that wants to split, never while that solve's stream is being captured.
//   scratch  the device address of this GPU's copy of the static workspace below.
constexpr int kSideStreams = 3;
struct Device {
    hipStream_t stream[kSideStreams] = {};
    hipEvent_t join[kSideStreams] = {};
    hipEvent_t fork = nullptr;
    hipEvent_t stagger = nullptr;
    bool helpers_tried = false, helpers_ok = false;
    void* scratch = nullptr;
    std::mutex busy;  // one fork/join sequence at a time per device
};

// Workspace of ckpt_solve_batched_noalloc, for callers that cannot allocate: a fixed array in
// every GPU's copy of the code object, held until the process ends.  In host code the array's
// name is only a handle for hipGetSymbolAddress; kernels are given the resolved address.
static __device__ __align__(256) unsigned char g_scratch[CKPT_NOALLOC_MAX_WORKSPACE + kScratchSlack];

std::mutex g_devices_lock;
Device g_devices[64];

Device* current_device() {
    int dev = 0;
    if (!hip_ok(hipGetDevice(&dev)) || dev < 0 || dev >= 64) return nullptr;
    return &g_devices[dev];
}

// Both set-up steps run with the device current and under g_devices_lock.
bool ensure_helpers(Device& d) {
    std::lock_guard<std::mutex> guard(g_devices_lock);
    if (!d.helpers_tried) {
        d.helpers_tried = true;
        bool ok = hip_ok(hipEventCreateWithFlags(&d.fork, hipEventDisableTiming)) &&
                  hip_ok(hipEventCreateWithFlags(&d.stagger, hipEventDisableTiming));
        for (int k = 0; k < kSideStreams && ok; ++k)
            ok = hip_ok(hipStreamCreateWithFlags(&d.stream[k], hipStreamNonBlocking)) &&
                 hip_ok(hipEventCreateWithFlags(&d.join[k], hipEventDisableTiming));
        d.helpers_ok = ok;
    }
    return d.helpers_ok;
}

// Resolves this device's address of g_scratch once (the device must be current).
void* ensure_scratch(Device& d) {
    std::lock_guard<std::mutex> guard(g_devices_lock);
    if (!d.scratch) {
        void* p = nullptr;
        if (!hip_ok(hipGetSymbolAddress(&p, HIP_SYMBOL(g_scratch))) || !p) return nullptr;
        d.scratch = p;
    }
    return d.scratch;
}

bool helpers_ready(Device& d) {
    std::lock_guard<std::mutex> guard(g_devices_lock);
    return d.helpers_ok;
}

// The frontier kernel keeps its triangle in LDS, chain_kernel its table; above the default per-block limit they have to be
// allowed the size.  Set once (to the largest size any L can need); allocates nothing.
bool allow_lds() {
    static std::once_flag once;
    static bool ok = false;
    std::call_once(once, [] {
        ok = hip_ok(hipFuncSetAttribute(reinterpret_cast<const void*>(frontier_kernel),
                                        hipFuncAttributeMaxDynamicSharedMemorySize,
                                        int(ckpt_table_rows(CKPT_MAX_L) * sizeof(int32_t))));
        for (const void* f : {reinterpret_cast<const void*>(chain_kernel<8>), reinterpret_cast<const void*>(chain_kernel<ckpt_rules::kChainStages>)})
            ok = ok && hip_ok(hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(ckpt_rules::kChainLds)));
    });
    return ok;
}

// Which kernels fill the table, and on how many streams.
//
// Several streams.  Chains are independent, so from D = 2 on the batch is split in up to four
// groups that run the same launch sequence on as many streams: the many short row launches
// of one group overlap with work of the others instead of leaving the machine idle between
// dependent launches.  The frontier kernel (a few busy CUs for a long time) runs on the first
// side stream beside everything else: the fill prunes with whatever frontier is in memory,
// the weak one of the precompute kernel or the exact one.  The side streams are forked from
// and joined back into the caller's stream with events.  Small problems are bound by launch
// latency, where more streams only add launches.
// Automatic choice: split when the batch is large enough to be bound by the GPU and not by
// launch latency (where more streams only add launches).  The caller can force either way.
struct Route {
    int groups;         // of chains, a stream each
    bool chain, flow;   // one launch: chain_kernel, or (behind precompute_kernel) flow_kernel
    bool flow_bounds;
};
Route route_of(int L, int pitch, int B, bool samples, const ckpt_solve_opts_t* opts) {
    const int nblk = blocks_of(L), want_groups = opts ? opts->groups : 0;
    const bool large = B >= 2 && size_t(B) * nblk * pitch >= (size_t(1) << 19);
    Route r{};
    r.groups = std::min(want_groups ? want_groups : (large ? kSideStreams + 1 : 1), B);
    if (nblk < 3) r.groups = 1;  // no diagonal to split
    // Small batches: every tile in one launch.  A schedule that the caller asks for is made of separate launches.
    const bool apart = opts && (opts->row_launches || opts->list_split);
    r.flow = r.groups == 1 && !apart && ckpt_rules::flow_pays(nblk, pitch / 64, B, samples);
    r.chain = !apart && !want_groups && !(opts && (opts->frontier || opts->spin_limit)) && ckpt_rules::chain_pays(L, pitch);
    r.flow_bounds = ckpt_rules::flow_bounds(nblk, pitch / 64, B, samples);
    return r;
}

int solve_impl(const ckpt_chains_t* chains, int L, int M, int B, void* stream, int32_t* cost, uint8_t* arg,
               void* workspace, size_t workspace_bytes, Profile* prof, const ckpt_solve_opts_t* opts,
               bool may_create_helpers) {
    if (!chains || !cost || !arg || !workspace) return CKPT_E_ARG;
    if (int rc = check_dims(L, M, B)) return rc;
    if (!chains->uf || !chains->ub || !chains->wa || !chains->wabar) return CKPT_E_ARG;
    if ((reinterpret_cast<uintptr_t>(cost) | reinterpret_cast<uintptr_t>(arg) |
         reinterpret_cast<uintptr_t>(workspace)) & 255)
        return CKPT_E_ARG;
    const int want_groups = opts ? opts->groups : 0, want_ks = opts ? opts->list_split : 0;
    const int row_mode = opts ? opts->row_launches : 0;
    if (row_mode != 0 && row_mode != 1) return CKPT_E_ARG;
    const bool fused_rows = row_mode == 0;
    const int stagger = opts ? opts->stagger : 0;
    const int frontier_mode = opts ? opts->frontier : 0;
    const int spin_limit = opts && opts->spin_limit ? opts->spin_limit : kSpinLimit;
    if (frontier_mode < 0 || frontier_mode > 2) return CKPT_E_ARG;
    unsigned long long* work = prof ? prof->work : nullptr;
    if (want_groups < 0 || want_groups > kSideStreams + 1) return CKPT_E_ARG;
    if (want_ks != 0 && want_ks != 1 && want_ks != 2 && want_ks != 4) return CKPT_E_ARG;
    bool own_side = false;
    if (opts) {
        for (int k = 0; k < kSideStreams; ++k) own_side = own_side || opts->side_streams[k];
        for (int k = 0; k < kSideStreams && own_side; ++k)
            if (!opts->side_streams[k] && k + 2 <= (want_groups ? want_groups : kSideStreams + 1)) return CKPT_E_ARG;
    }
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int pitch = int(ckpt_row_pitch(M));
    const int rows = int(ckpt_table_rows(L));
    // without room for the samples (the static workspace of the entry point that allocates nothing) the
    // block product evaluates every feasible split
    const Workspace ws = carve(workspace, L, pitch, B, workspace_bytes >= ckpt_workspace_bytes(L, M, B));

    const size_t frontier_lds = ckpt_table_rows(L) * sizeof(int32_t);
    if (frontier_lds > 48 * 1024 && !allow_lds()) return CKPT_E_HIP;
    constexpr int T = kT;
    const int nblk = (L + T - 1) / T;
    const int gx_row = (pitch + kRowWG - 1) / kRowWG;

    const Route route = route_of(L, pitch, B, ws.samp, opts);
    const bool chain = route.chain, flow = route.flow;
    int groups = route.groups;
    const bool would_split = groups > 1;
    const size_t chain_lds = ckpt_rules::chain_lds(L, pitch);
    if (chain && chain_lds > 48 * 1024 && !allow_lds()) return CKPT_E_HIP;
    if (prof) groups = 1;  // the event trail times one stream
    Device* dev = nullptr;
    if (groups > 1) {
        dev = current_device();
        if (!dev) return CKPT_E_HIP;
        if (!helpers_ready(*dev)) {
            // Streams and events are not created behind a capture: a captured stream must only see
            // enqueued work.  ckpt_init beforehand makes the split available to captured solves.
            hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
            if (!hip_ok(hipStreamIsCapturing(st, &cap))) return CKPT_E_HIP;
            if (cap != hipStreamCaptureStatusNone || !may_create_helpers) {
                if (want_groups > 1) return CKPT_E_NOTREADY;
                groups = 1;
            } else if (!ensure_helpers(*dev)) {
                return CKPT_E_HIP;
            }
        }
    }
    Device* side = groups > 1 ? dev : nullptr;
    // The exact frontier costs one long single-block launch per chain, 0.05 to 0.65 ms from 96 to 254 stages whatever
    // the batch.  On a side stream it runs beside the fill (64 x 96 stages 3.29 ms, 3.43 without it; 8 x 192 stages
    // 4.04 and 4.26; of 19 shapes only 2 x 254 stages at 8192 slots are slower with it, 4.60 and 4.48).  On the caller's
    // stream it pays only when the pruning it adds saves more than it costs.  Both grow with the length of the
    // chains, so the line is one of width, columns x blocks of stages: one stream, 4 x 254 stages and 1500 slots
    // (2.0e5 by that measure) 3.32 ms with it, 2.68 without; 3 x 192, 4096 slots (3.0e5) 2.50 and 2.20; 8 x 254, 1000
    // slots (2.6e5) 3.82 and 3.23; 6 x 192, 4096 slots (6.0e5) 3.81 and 3.65; 7 x 254, 4096 slots (9.3e5) 7.60 and 7.57;
    // 1 x 192, 40000 slots (9.6e5) 5.36 and 5.58; 10 x 192, 4096 slots (10.0e5) 5.36 and 5.42; 60 x 64, 2048 slots
    // (10.1e5) 1.36 and 1.38; 64 x 96, 2048 slots (16e5) 3.57 and 3.63; 12 x 254, 4096 slots (16e5) 11.3 and 11.9.
    // Chains of few blocks have little to prune: 40 x 60 stages (5.4e6 by columns x blocks^2) 942 us and 944.
    const bool wide = size_t(B) * pitch * nblk >= 950000 && size_t(B) * pitch * nblk * nblk >= 6000000;
    // A profiled solve runs the kernels that the automatic schedule would run, on one stream.
    const bool beside = groups > 1 || (prof && would_split);
    const bool want_frontier = frontier_mode == 1 || (frontier_mode == 0 && (beside || wide));
    std::unique_lock<std::mutex> lock;
    if (side) lock = std::unique_lock<std::mutex>(side->busy);  // one fork/join at a time per device
    hipStream_t gs[kSideStreams + 1] = {st, st, st, st};  // stream of group g
    hipStream_t side_stream[kSideStreams] = {};
    for (int g = 1; g < groups; ++g)
        gs[g] = side_stream[g - 1] = own_side ? static_cast<hipStream_t>(opts->side_streams[g - 1]) : side->stream[g - 1];
    int first[kSideStreams + 2];  // group g holds chains first[g] .. first[g + 1] - 1
    for (int g = 0; g <= groups; ++g) first[g] = int((long long)B * g / groups);

    int forked = 0;  // side streams that wait on the caller's stream and have to be joined back
    auto join_side = [&](int k) {  // the caller's stream waits for side stream k
        return hip_ok(hipEventRecord(side->join[k], side_stream[k])) &&
               hip_ok(hipStreamWaitEvent(st, side->join[k], 0));
    };
    auto enqueue = [&]() -> int {
        if (chain) {
            hipLaunchKernelGGL(L <= 8 ? chain_kernel<8> : chain_kernel<ckpt_rules::kChainStages>, dim3(B), dim3(pitch), chain_lds, st, *chains, L,
                               pitch, ws, cost, arg, work);
            CKPT_AFTER_LAUNCH(CKPT_K_ROW);
            return CKPT_OK;
        }
        const int pre_rows = ckpt_rules::precompute_rows(L, B), pre_parts = (L + pre_rows - 1) / pre_rows;
        const int mark_parts = flow ? nblk * ((pitch + kMarkCols - 1) / kMarkCols) : 0;
        hipLaunchKernelGGL(precompute_kernel, dim3(B, pre_parts + 1 + mark_parts), dim3(flow ? kPreThreads : (L + 63) / 64 * 64), 0, st,
                           *chains, L, pitch, ws, pre_rows, pre_parts, cost);
        CKPT_AFTER_LAUNCH(CKPT_K_PRECOMPUTE);
        if (side) {
            if (!hip_ok(hipEventRecord(side->fork, st)) || !hip_ok(hipStreamWaitEvent(gs[1], side->fork, 0)))
                return CKPT_E_HIP;
            forked = 1;
        }
        if (want_frontier) {
            hipLaunchKernelGGL(frontier_kernel, dim3(B), dim3(1024), frontier_lds, gs[1], *chains, L, ws);
            CKPT_AFTER_LAUNCH(CKPT_K_FRONTIER);
        }

        if (flow) {
            const Ctx ctx{L, M, pitch, rows, 0, spin_limit, ws, cost, arg, work, false};
            hipLaunchKernelGGL(route.flow_bounds ? flow_kernel<true> : flow_kernel<false>, dim3(unsigned(tiles_of(L) * (pitch / 64) * B)), dim3(kFlow), 0, st, ctx, B);
            CKPT_AFTER_LAUNCH(CKPT_K_ROW);
            return CKPT_OK;
        }
        const int nbands = bands_of(pitch);
        for (int D = 0; D < 2 && D < nblk; ++D) {
            const Ctx ctx{L, M, pitch, rows, 0, spin_limit, ws, cost, arg, work, false};
            if (fused_rows) {
                const dim3 grid(nbands, nblk - D, B);
                const auto fn = D == 0 ? (work ? tile_rows_kernel<0, true> : tile_rows_kernel<0, false>)
                                       : (work ? tile_rows_kernel<1, true> : tile_rows_kernel<1, false>);
                hipLaunchKernelGGL(fn, grid, dim3(kRowWG), 0, st, ctx, D);
                CKPT_AFTER_LAUNCH(CKPT_K_ROW);
                continue;
            }
            const auto& rowfn = D == 0 ? kRow0 : kRow1;
            for (int r = T - 1; r >= 0; --r) {
                hipLaunchKernelGGL(rowfn[r], dim3(gx_row, nblk - D, B), dim3(kRowWG), 0, st, ctx, D);
                CKPT_AFTER_LAUNCH(CKPT_K_ROW);
            }
        }
        if (side) {
            // every side stream waits for the D < 2 rows.  Nobody waits for the frontier kernel: the
            // fill uses whatever frontier is in memory, and the group on its stream follows it anyway.
            if (!hip_ok(hipEventRecord(side->fork, st))) return CKPT_E_HIP;
            for (int g = 1; g < groups; ++g) {
                if (!hip_ok(hipStreamWaitEvent(gs[g], side->fork, 0))) return CKPT_E_HIP;
                forked = g;
            }
        }
        for (int D = 2; D < nblk; ++D) {
            // Later diagonals have fewer tiles and longer work lists.  The chip holds 2048 chunks (of two
            // waves each); a launch with few of them leaves it half empty while the last ones finish, so 2 or 4
            // slices of waves share a chunk.  That pays only with splits to share, 8 (D - 1) + 1 of them in
            // passes of 16: 8 x 192 stages gain 2 % up to 7000 chunks (D = 11), while with 5000 chunks at D = 4
            // (40 x 60 stages) or 2000 at D = 3 (30 x 32) a list for one slice is 3.5 % faster a solve; at D = 4, with
            // two passes, 4 slices cost 16 x 48 stages 3 % against 2.  4 slices up to 600, 800 and 1100 chunks: 3 x 254 stages
            // 2186, 2154 and 2138 us, 1 x 192 1162, 1135 and 1133, 20 x 80 419, 425 and 432, 8 x 128 774, 771 and 781,
            // 8 x 96, 2048 slots 654, 654 and 660.
            const long long chunks = (long long)(nblk - D) * (pitch / 64) * B;
            const int ks = want_ks ? want_ks : (chunks <= 800 && D >= 5 ? 4 : (chunks <= 600 * D ? 2 : 1));
            const int ch = ks == 1 ? kCH : 1, halves = halves_of(ks), gx = (pitch / 64 + ch - 1) / ch * (2 / halves);
            const bool passing = beside && ckpt_rules::rows_pass(nblk - D, pitch, B);
            for (int g = 0; g < groups; ++g) {
                const Ctx ctx{L, M, pitch, rows, first[g], spin_limit, ws, cost, arg, work, passing};
                const dim3 grid(gx, nblk - D, first[g + 1] - first[g]), block(64 * halves * ch * ks);
                const auto fn = ks == 4 ? (work ? gemm_kernel<1, 4, true> : gemm_kernel<1, 4, false>)
                              : ks == 2 ? (work ? gemm_kernel<1, 2, true> : gemm_kernel<1, 2, false>)
                                        : (work ? gemm_kernel<kCH, 1, true> : gemm_kernel<kCH, 1, false>);
                hipLaunchKernelGGL(fn, grid, block, 0, gs[g], ctx, D);
                CKPT_AFTER_LAUNCH(CKPT_K_GEMM);
                if (D == 2 && g == 0 && side && stagger && groups >= 3) {
                    // the second half of the groups starts when the first group's block product is
                    // done: from then on their bandwidth-bound and latency-bound phases alternate
                    if (!hip_ok(hipEventRecord(side->stagger, gs[0]))) return CKPT_E_HIP;
                    for (int h = (groups + 1) / 2; h < groups; ++h)
                        if (!hip_ok(hipStreamWaitEvent(gs[h], side->stagger, 0))) return CKPT_E_HIP;
                }
            }
            if (fused_rows) {  // rows 6..0 of every tile of the diagonal in one launch per group
                for (int g = 0; g < groups; ++g) {
                    const Ctx ctx{L, M, pitch, rows, first[g], spin_limit, ws, cost, arg, work, false};
                    const auto fn = work ? tile_rows_kernel<2, true> : tile_rows_kernel<2, false>;
                    hipLaunchKernelGGL(fn, dim3(nbands, nblk - D, first[g + 1] - first[g]), dim3(kRowWG), 0, gs[g], ctx, D);
                    CKPT_AFTER_LAUNCH(CKPT_K_ROW);
                }
                continue;
            }
            // rows of the groups are issued in turn so that every queue stays fed; row 7 was
            // finished by the gemm
            for (int r = T - 2; r >= 0; --r) {
                for (int g = 0; g < groups; ++g) {
                    const Ctx ctx{L, M, pitch, rows, first[g], spin_limit, ws, cost, arg, work, false};
                    hipLaunchKernelGGL(kRow2[r], dim3(gx_row, nblk - D, first[g + 1] - first[g]), dim3(kRowWG), 0,
                                       gs[g], ctx, D);
                    CKPT_AFTER_LAUNCH(CKPT_K_ROW);
                }
            }
        }
        return CKPT_OK;
    };
    int rc = enqueue();
    // Every forked side stream rejoins the caller's stream, also after a failed launch, so that
    // the caller's stream (or a capture in progress) is never left with an open fork.
    for (int k = 0; k < forked; ++k)
        if (!join_side(k) && rc == CKPT_OK) rc = CKPT_E_HIP;
    return rc;
}

}  // namespace

extern "C" {

size_t ckpt_workspace_bytes(int L, int M, int B) {
    if (L < 1 || M < 0 || B < 1) return 0;
    const int pitch = int(ckpt_row_pitch(M));
    const size_t samples = uses_bounds(L, pitch, B) ? size_t(B) * samp_ints(L, pitch) : 0;
    return (ws_ints(L, pitch, B) + samples) * sizeof(int32_t);
}

// Whether the static workspace has room for what a solve cannot do without (everything but the samples).
static bool fits_static_workspace(int L, int M, int B) {
    const int pitch = int(ckpt_row_pitch(M));
    return limit_ints(L, pitch, B) * sizeof(int32_t) <= CKPT_NOALLOC_MAX_WORKSPACE &&
           ws_ints(L, pitch, B) * sizeof(int32_t) <= sizeof(g_scratch);
}

int ckpt_init(int device) {
    if (device >= 64) return CKPT_E_LIMIT;
    int prev = 0;
    if (!hip_ok(hipGetDevice(&prev))) return CKPT_E_HIP;
    if (device < 0) device = prev;
    if (device >= 64) return CKPT_E_LIMIT;
    if (device != prev && !hip_ok(hipSetDevice(device))) return CKPT_E_HIP;
    Device& d = g_devices[device];
    const bool ok = ensure_helpers(d) && ensure_scratch(d) != nullptr && allow_lds();
    if (device != prev && !hip_ok(hipSetDevice(prev))) return CKPT_E_HIP;
    return ok ? CKPT_OK : CKPT_E_HIP;
}

int ckpt_solve_batched(const ckpt_chains_t* chains, int L, int M, int B, void* stream, int32_t* cost,
                       uint8_t* arg, void* workspace) {
    return solve_impl(chains, L, M, B, stream, cost, arg, workspace, ~size_t(0), nullptr, nullptr, true);
}

int ckpt_solve_batched_noalloc(const ckpt_chains_t* chains, int L, int M, int B, void* stream, int32_t* cost,
                               uint8_t* arg) {
    if (int rc = check_dims(L, M, B)) return rc;
    if (!fits_static_workspace(L, M, B)) return CKPT_E_LIMIT;
    Device* dev = current_device();
    if (!dev) return CKPT_E_HIP;
    void* scratch = ensure_scratch(*dev);
    if (!scratch) return CKPT_E_HIP;
    // creates nothing: the batch is split only if the helper streams exist already
    return solve_impl(chains, L, M, B, stream, cost, arg, scratch, CKPT_NOALLOC_MAX_WORKSPACE, nullptr, nullptr, false);
}

int ckpt_solve_batched_opts(const ckpt_chains_t* chains, int L, int M, int B, void* stream, int32_t* cost,
                            uint8_t* arg, void* workspace, const ckpt_solve_opts_t* opts) {
    return solve_impl(chains, L, M, B, stream, cost, arg, workspace, ~size_t(0), nullptr, opts, true);
}

int ckpt_solve_profiled(const ckpt_chains_t* chains, int L, int M, int B, void* stream, int32_t* cost,
                        uint8_t* arg, void* workspace, float* kind_ms, int* kind_launches, double* kind_bytes) {
    if (!kind_ms || !kind_launches) return CKPT_E_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    Profile prof;
    prof.stream = st;
    for (int k = 0; k < CKPT_N_KERNEL_KINDS; ++k) kind_ms[k] = 0.f, kind_launches[k] = 0;
    int rc = CKPT_OK;
    if (!prof.mark(-1)) rc = CKPT_E_HIP;
    if (rc == CKPT_OK) rc = solve_impl(chains, L, M, B, stream, cost, arg, workspace, ~size_t(0), &prof, nullptr, false);
    if (!hip_ok(hipStreamSynchronize(st)) && rc == CKPT_OK) rc = CKPT_E_HIP;
    for (size_t i = 1; i < prof.events.size() && rc == CKPT_OK; ++i) {
        float ms = 0.f;
        if (!hip_ok(hipEventElapsedTime(&ms, prof.events[i - 1], prof.events[i]))) rc = CKPT_E_HIP;
        kind_ms[prof.kinds[i]] += ms;
        kind_launches[prof.kinds[i]] += 1;
    }
    for (hipEvent_t e : prof.events) (void)hipEventDestroy(e);
    if (kind_bytes && rc == CKPT_OK) {
        // a second, untimed pass in which every wave adds up the bytes it asks for
        for (int k = 0; k < 2 * CKPT_N_KERNEL_KINDS; ++k) kind_bytes[k] = 0.0;
        Profile count;
        count.stream = st;
        count.trail = false;
        std::vector<unsigned long long> host(size_t(kWorkSets) * 4, 0);
        const size_t bytes = host.size() * sizeof(unsigned long long);
        if (!hip_ok(hipMalloc(reinterpret_cast<void**>(&count.work), bytes))) return CKPT_E_HIP;
        if (!hip_ok(hipMemsetAsync(count.work, 0, bytes, st))) rc = CKPT_E_HIP;
        if (rc == CKPT_OK) rc = solve_impl(chains, L, M, B, stream, cost, arg, workspace, ~size_t(0), &count, nullptr, false);
        if (rc == CKPT_OK && !hip_ok(hipMemcpyAsync(host.data(), count.work, bytes, hipMemcpyDeviceToHost, st)))
            rc = CKPT_E_HIP;
        if (!hip_ok(hipStreamSynchronize(st)) && rc == CKPT_OK) rc = CKPT_E_HIP;
        (void)hipFree(count.work);
        for (int set = 0; set < kWorkSets; ++set) {
            kind_bytes[2 * CKPT_K_GEMM] += double(host[set * 4]);
            kind_bytes[2 * CKPT_K_GEMM + 1] += double(host[set * 4 + 1]);
            kind_bytes[2 * CKPT_K_ROW] += double(host[set * 4 + 2]);
            kind_bytes[2 * CKPT_K_ROW + 1] += double(host[set * 4 + 3]);
        }
    }
    return rc;
}

const char* ckpt_kernel_name(int kind) {
    switch (kind) {
        case CKPT_K_PRECOMPUTE: return "precompute_kernel";
        case CKPT_K_FRONTIER: return "frontier_kernel";
        case CKPT_K_GEMM: return "gemm_kernel";
        case CKPT_K_ROW: return "tile_rows_kernel";
        default: return nullptr;
    }
}

const char* ckpt_kernel_name_of(int kind, int L, int M, int B) {
    if (kind == CKPT_K_ROW && check_dims(L, M, B) == CKPT_OK) {
        const int pitch = int(ckpt_row_pitch(M));
        const Route route = route_of(L, pitch, B, samples_of(L, pitch, B), nullptr);
        if (route.chain) return "chain_kernel";
        if (route.flow) return "flow_kernel";
    }
    return ckpt_kernel_name(kind);
}

int ckpt_check_inputs(const void* workspace, int L, int M, int B, void* stream, int32_t* flags_host) {
    if (!flags_host) return CKPT_E_ARG;
    if (int rc = check_dims(L, M, B)) return rc;
    if (!workspace) {  // the static workspace of ckpt_solve_batched_noalloc on the current device
        if (!fits_static_workspace(L, M, B)) return CKPT_E_LIMIT;
        Device* dev = current_device();
        workspace = dev ? ensure_scratch(*dev) : nullptr;
        if (!workspace) return CKPT_E_HIP;
    }
    const Workspace ws = carve(const_cast<void*>(workspace), L, int(ckpt_row_pitch(M)), B, false);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (!hip_ok(hipMemcpyAsync(flags_host, ws.flags, size_t(B) * sizeof(int32_t), hipMemcpyDeviceToHost, st)))
        return CKPT_E_HIP;
    int32_t fault = 0;
    if (!hip_ok(hipMemcpyAsync(&fault, ws.fault, sizeof(int32_t), hipMemcpyDeviceToHost, st))) return CKPT_E_HIP;
    if (!hip_ok(hipStreamSynchronize(st))) return CKPT_E_HIP;
    if (fault) return CKPT_E_INTERNAL;
    for (int b = 0; b < B; ++b)
        if (flags_host[b]) return CKPT_E_INPUT;
    return CKPT_OK;
}

int ckpt_select_plan(const int32_t* cost, int L, int M, int B, const int32_t* m_budget, void* stream,
                     int32_t* out) {
    if (!cost || !m_budget || !out) return CKPT_E_ARG;
    if (int rc = check_dims(L, M, B)) return rc;
    hipLaunchKernelGGL(select_kernel, dim3(1), dim3(256), 0, static_cast<hipStream_t>(stream), cost, L, M,
                       int(ckpt_row_pitch(M)), int(ckpt_table_rows(L)), B, m_budget, out);
    return hip_ok(hipGetLastError()) ? CKPT_OK : CKPT_E_HIP;
}

int ckpt_discretize(const int64_t* bytes_wa, const int64_t* bytes_wabar, const int64_t* bytes_wdelta,
                    const int64_t* bytes_of, const int64_t* bytes_ob, const int64_t* budget_bytes, int L,
                    int M, int B, void* stream, const ckpt_chains_t* out) {
    if (!bytes_wa || !bytes_wabar || !budget_bytes || !out || !out->wa || !out->wabar) return CKPT_E_ARG;
    if ((bytes_wdelta && !out->wdelta) || (bytes_of && !out->of) || (bytes_ob && !out->ob)) return CKPT_E_ARG;
    if (int rc = check_dims(L, M, B)) return rc;
    if (M > (1 << 20)) return CKPT_E_LIMIT;
    hipStream_t st = static_cast<hipStream_t>(stream);
    struct Job { const int64_t* in; const int32_t* out; int n; };
    const Job jobs[5] = {{bytes_wa, out->wa, L + 1}, {bytes_wabar, out->wabar, L}, {bytes_wdelta, out->wdelta, L + 1},
                         {bytes_of, out->of, L}, {bytes_ob, out->ob, L}};
    for (const Job& j : jobs) {
        if (!j.in) continue;
        hipLaunchKernelGGL(discretize_kernel, dim3((j.n + 255) / 256, B), dim3(256), 0, st,
                           reinterpret_cast<const long long*>(j.in), const_cast<int32_t*>(j.out),
                           reinterpret_cast<const long long*>(budget_bytes), j.n, M);
        if (!hip_ok(hipGetLastError())) return CKPT_E_HIP;
    }
    return CKPT_OK;
}

int ckpt_discretize_sweep(const int64_t* bytes_wa, const int64_t* bytes_wabar, const int64_t* bytes_wdelta,
                          const int64_t* bytes_of, const int64_t* bytes_ob, int64_t base_budget, int alpha_num,
                          int alpha_den, int count, int L, int M, void* stream, int64_t* budgets_out,
                          const ckpt_chains_t* out) {
    if (!bytes_wa || !bytes_wabar || !out || !out->wa || !out->wabar) return CKPT_E_ARG;
    if ((bytes_wdelta && !out->wdelta) || (bytes_of && !out->of) || (bytes_ob && !out->ob)) return CKPT_E_ARG;
    SweepBudgets budget{};
    static_assert(sizeof(long long) == sizeof(int64_t), "budget words");
    if (int rc = ckpt_budget_sweep(base_budget, alpha_num, alpha_den, count, reinterpret_cast<int64_t*>(budget.v)))
        return rc;
    if (int rc = check_dims(L, M, count)) return rc;
    if (M > (1 << 20)) return CKPT_E_LIMIT;
    hipStream_t st = static_cast<hipStream_t>(stream);
    SweepArrays arrays{};
    int n = 0;
    auto add = [&](const int64_t* in, const int32_t* to, int per_chain) {
        if (in) arrays.v[n++] = SweepArray{in, const_cast<int32_t*>(to), per_chain};
    };
    add(bytes_wa, out->wa, L + 1), add(bytes_wabar, out->wabar, L), add(bytes_wdelta, out->wdelta, L + 1);
    add(bytes_of, out->of, L), add(bytes_ob, out->ob, L);
    hipLaunchKernelGGL(discretize_sweep_kernel, dim3(n + (budgets_out ? 1 : 0), count), dim3(kSweepThreads), 0, st, arrays, n, budget, count,
                       reinterpret_cast<long long*>(budgets_out), M);
    return hip_ok(hipGetLastError()) ? CKPT_OK : CKPT_E_HIP;
}

size_t ckpt_schedule_workspace_bytes(int L, int B) {
    if (L < 1 || B < 1) return 0;
    return size_t(B) * (2 * size_t(L) + 2) * sizeof(int4);
}

int ckpt_schedule_batched(const uint8_t* arg, const int32_t* wa, const int32_t* wabar, int L, int M, int B,
                          const int32_t* m_budget, void* stream, ckpt_op_t* ops, int ops_cap, int32_t* n_ops,
                          void* workspace) {
    if (!arg || !wa || !wabar || !m_budget || !ops || !n_ops || !workspace || ops_cap < 0) return CKPT_E_ARG;
    if (reinterpret_cast<uintptr_t>(workspace) & 15) return CKPT_E_ARG;
    if (int rc = check_dims(L, M, B)) return rc;
    hipLaunchKernelGGL(schedule_kernel, dim3(B), dim3(kWalkThreads), 0, static_cast<hipStream_t>(stream), arg, wa, wabar,
                       L, M, int(ckpt_row_pitch(M)), int(ckpt_table_rows(L)), m_budget, ops, ops_cap, n_ops);
    return hip_ok(hipGetLastError()) ? CKPT_OK : CKPT_E_HIP;
}

int ckpt_block_indices_batched(const ckpt_op_t* ops, int ops_cap, const int32_t* n_ops, int L, int B, void* stream,
                               int32_t* block_of_stage, int32_t* n_blocks) {
    if (!ops || !n_ops || !block_of_stage || !n_blocks || ops_cap < 0 || L < 1 || B < 1) return CKPT_E_ARG;
    if (L > CKPT_MAX_L) return CKPT_E_LIMIT;
    hipLaunchKernelGGL(block_index_kernel, dim3(B), dim3(kBlockThreads), 0, static_cast<hipStream_t>(stream), ops, ops_cap, n_ops,
                       L, block_of_stage, n_blocks);
    return hip_ok(hipGetLastError()) ? CKPT_OK : CKPT_E_HIP;
}

int ckpt_simulate_batched(const ckpt_chains_t* chains, int L, int B, const ckpt_op_t* ops, int ops_cap,
                          const int32_t* n_ops, void* stream, int64_t* time_out, int64_t* peak_out,
                          int32_t* status) {
    if (!chains || !chains->uf || !chains->ub || !chains->wa || !chains->wabar || !ops || !n_ops || !time_out ||
        !peak_out || !status || ops_cap < 0 || L < 1 || B < 1)
        return CKPT_E_ARG;
    if (L > CKPT_MAX_L) return CKPT_E_LIMIT;
    hipLaunchKernelGGL(simulate_kernel, dim3(B), dim3(kSimThreads), 0, static_cast<hipStream_t>(stream), *chains, L, ops,
                       ops_cap, n_ops, reinterpret_cast<long long*>(time_out), reinterpret_cast<long long*>(peak_out),
                       status);
    return hip_ok(hipGetLastError()) ? CKPT_OK : CKPT_E_HIP;
}

int ckpt_last_hip_error(void) { return g_last_hip_error.load(); }


}  // extern "C"

// gfx950 kernel of the Interval Head's two linear maps (Sec. 3.2.1, "Interval Head Architecture": the head's
// output dimension is 2 |V|; c_t = Linear_center(h_t), raw radius = Linear_radius(h_t)):
//   out[n, j] = sum_k hidden[n, k] * weight[j, k] + bias[j],   j in [0, 2V)
// bf16 operands, fp32 accumulation on the matrix cores (v_mfma_f32_32x32x16_bf16), fp32 logits out: columns
// [0, V) go to the centre rows, [V, 2V) to the raw-radius rows, which the tensor-radius quantifier reads next.
#include <mutex>
#include "ciar_device.h"
#include <hip/hip_ext.h>

namespace ciar {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// Workgroup tile (64 MB) x (64 NB) x 64 with four waves in a 2 x 2 grid, each wave (32 MB) x (32 NB) = MB x NB MFMA
// blocks of 32 x 32.  MB = NB = 4 (256 x 256, a wave 128 x 128) is the shape for real vocabularies: a wave then
// reads 8 operand vectors from LDS for 16 matrix instructions, half the LDS traffic per instruction of the
// 128 x 128 tile (MB = NB = 2), which serves 33 to 128 rows, and up to 256 of vocabularies that are an odd multiple of 128.
// Measured (2048 rows, V = 16384): D = 1280 202 -> 192 us, D = 4096 510 -> 463 us when the requests moved between the matrix
// instructions of the fourth slice and the epilogue lost its barriers.
//
// Operand tiles go from memory straight into LDS (global_load_lds_dwordx4: no staging registers, and a request
// has a whole tile's multiplication to arrive in).  One such instruction writes the 64 lanes'
// 16-byte chunks to 1 KiB of consecutive LDS, i.e. eight tile rows of 64 bf16 without padding, so the chunks of a
// row are stored in swizzled order instead: chunk q of row r sits at position q ^ ((r / 2) % 8).  The lanes choose which
// chunk of their row they request accordingly (the eight lanes of a row still cover its 128 bytes), and the 32
// rows that one operand read touches at the same k are spread over the banks: a row is 32 banks wide, so the
// even rows share one half of the 64 banks and the odd rows the other, and any 16 consecutive rows (eight of
// each kind, with eight different positions) cover every bank once.
constexpr int BK = kHeadTileDepth;
constexpr int ROWB = BK * 2;            // bytes of a tile row in LDS
static_assert(BK == 64, "a tile row is eight 16-byte chunks");
using gptr = const __attribute__((address_space(1))) void*;
using lptr = __attribute__((address_space(3))) void*;

// Joins the workgroup's barrier when this wave's LDS operations are done (requests under way are not waited for).
__device__ __forceinline__ void lds_join() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Lane layout of v_mfma_f32_32x32x16_bf16: lane l supplies row (A) / column (B) l % 32 with the eight consecutive k
// 8 (l / 32) .. + 7; accumulator register v of lane l is the element (8 (v / 4) + 4 (l / 32) + v % 4, l % 32).
template <int MB, int NB>
__global__ __launch_bounds__(256) void interhead_gemm_kernel(const HeadArgs A)
{
    constexpr int BM = 64 * MB, BN = 64 * NB;
    constexpr int CA = BM / 32, CB = BN / 32;                      // load instructions per wave and tile (8 rows each)
    constexpr int BUF = (BM + BN) * ROWB;                          // bytes of one buffer: the A tile, then the B tile
    extern __shared__ __attribute__((aligned(1024))) char lds[];   // two buffers

    // (the wave's index in a scalar register, and with it the LDS addresses of its requests)
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    // Workgroups are handed to the eight XCDs in turn (workgroup b runs on XCD b % 8), and every XCD has an L2 of its
    // own.  So the tiles are dealt by XCD: XCD x takes the column tiles x, x + 8, ..., and its consecutive
    // workgroups walk the row tiles of one column tile.  The workgroups that are resident on an XCD together then
    // share their weight tile (and the few row tiles of hidden states) in that L2.
    int rt, ct;
    if (A.col_tiles % 8 == 0) {
        const int x = (int)(blockIdx.x & 7), local = (int)(blockIdx.x >> 3);
        rt = local % A.row_tiles;
        ct = (local / A.row_tiles) * 8 + x;
    } else {
        rt = (int)(blockIdx.x % A.row_tiles);
        ct = (int)(blockIdx.x / A.row_tiles);
    }
    const int64_t m0 = (int64_t)rt * BM;
    const int n0 = ct * BN;                                        // column of the 2V-wide output

    // Requests: instruction u of wave w covers the tile rows 8 (w + 4 u) .. + 7; lane l asks for row + l / 8 and,
    // of that row, the chunk that belongs at position l % 8.  Addresses: a uniform base per tile plus one 32-bit
    // byte offset per instruction (rows past the end of the batch repeat the last row; they are never stored).
    uint32_t oa[CA], ob[CB];
    const int rl = lane >> 3, chunk = (lane & 7) ^ ((4 * (wave & 1)) | (rl >> 1));   // row = 8 (w + 4 u) + rl: (row / 2) % 8
    const int64_t last = A.N - 1 - m0;                             // >= 0: the tile starts inside the batch
#pragma unroll
    for (int u = 0; u < CA; ++u) {
        const int row = 8 * (wave + 4 * u) + rl;
        oa[u] = (uint32_t)(row <= last ? row : (int)last) * (uint32_t)A.D * 2u + (uint32_t)chunk * 16u;
    }
#pragma unroll
    for (int u = 0; u < CB; ++u) ob[u] = (uint32_t)(8 * (wave + 4 * u) + rl) * (uint32_t)A.D * 2u + (uint32_t)chunk * 16u;
    const gbytes baseA = (gbytes)(A.hidden + m0 * A.D), baseB = (gbytes)(A.weight + (int64_t)n0 * A.D);
    // (the bases through an empty asm: a request is then one load from a scalar base and a 32-bit lane offset, not a 64-bit
    // address per lane and request)
    uint64_t kA, kB;
    int dst;
    auto request_from = [&](int k0, int buf) {
        kA = (uint64_t)baseA + (uint32_t)k0 * 2u;
        kB = (uint64_t)baseB + (uint32_t)k0 * 2u;
        dst = buf * BUF + wave * 8 * ROWB;
        asm volatile("" : "+s"(kA), "+s"(kB));
    };
    auto request_one = [&](int u) {
        if (u < CA) __builtin_amdgcn_global_load_lds((gptr)((gbytes)kA + oa[u < CA ? u : 0]), (lptr)(lds + dst + u * 32 * ROWB), 16, 0, 0);
        else __builtin_amdgcn_global_load_lds((gptr)((gbytes)kB + ob[u < CA ? 0 : u - CA]),
                                              (lptr)(lds + dst + BM * ROWB + (u - CA) * 32 * ROWB), 16, 0, 0);
    };
    auto request = [&](int k0, int buf) {
        request_from(k0, buf);
#pragma unroll
        for (int u = 0; u < CA + CB; ++u) request_one(u);
    };

    f32x16 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // Operand reads: lane l reads row l % 32 of each 32-row block; its chunk in slice sl (k 16 sl .. + 15) is
    // 2 sl + l / 32, stored at position (2 sl) ^ sw with sw = (l / 32) ^ ((row / 2) % 8).
    const int lrow = lane & 31, sw = (lane >> 5) ^ ((lrow >> 1) & 7);
    const int offA = (wm * 32 * MB + lrow) * ROWB, offB = BM * ROWB + (wn * 32 * NB + lrow) * ROWB;

    // Pipeline over the k tiles, one barrier per tile.  A tile is multiplied in four 16-deep slices; the operands
    // of a slice are read from LDS during the matrix instructions of the slice before (two register sets), early in
    // it, so that a slice never starts by waiting for LDS.  The barrier stands after the third slice: by then every
    // wave holds its last operands of the current tile in registers, so behind the barrier the tile's buffer is
    // free and the tile after the next is requested into it at once, a whole tile's multiplication ahead of its
    // use; the fourth slice already reads the first operands of the next tile, whose arrival the barrier has
    // awaited (own requests, then the other waves).  Past the last tile the requests repeat it, so no branch
    // splits the loop body; the barrier before the epilogue awaits the last of them.
    static_assert(MB == NB && BK == 64, "the slice pattern below is written for square wave tiles, four slices");
    const int klast = A.D - BK;
    bf16x8 a[2][MB], b[2][NB];
    auto operands = [&](const char* tile, int sl, int set) {
        const int pos = ((2 * sl) ^ sw) * 16;
#pragma unroll
        for (int i = 0; i < MB; ++i) a[set][i] = *reinterpret_cast<const bf16x8*>(tile + offA + i * 32 * ROWB + pos);
#pragma unroll
        for (int j = 0; j < NB; ++j) b[set][j] = *reinterpret_cast<const bf16x8*>(tile + offB + j * 32 * ROWB + pos);
    };
    auto multiply = [&](int set) {
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
            for (int j = 0; j < NB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[set][i], b[set][j], acc[i][j], 0, 0, 0);
    };
    // one LDS read after each of the first MB + NB matrix instructions of a slice, the rest of the slice without
    auto pattern = [&]() {
#pragma unroll
        for (int g = 0; g < MB + NB; ++g) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);     // a matrix instruction
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);     // an LDS read
        }
        __builtin_amdgcn_sched_group_barrier(0x008, MB * NB - (MB + NB), 0);
    };
    // The fourth slice, written out: behind each matrix instruction one LDS read (the next tile's first operands) while there are
    // any, and a request or two.  (One behind another the requests hold the matrix pipe up for ~400 cycles a tile.)
    auto last_slice = [&](const char* nxt) {
        constexpr int PER = (CA + CB + MB * NB - 1) / (MB * NB), READS = (MB + NB + MB * NB - 1) / (MB * NB);
        const int pos = sw * 16;
#pragma unroll
        for (int g = 0; g < MB * NB; ++g) {
            const int i = g / NB, j = g % NB;
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1][i], b[1][j], acc[i][j], 0, 0, 0);
#pragma unroll
            for (int q = g * READS; q < (g + 1) * READS; ++q) {
                if (q < MB) a[0][q < MB ? q : 0] = *reinterpret_cast<const bf16x8*>(nxt + offA + q * 32 * ROWB + pos);
                else if (q < MB + NB) b[0][q < MB ? 0 : (q - MB < NB ? q - MB : 0)] = *reinterpret_cast<const bf16x8*>(nxt + offB + (q - MB) * 32 * ROWB + pos);
            }
#pragma unroll
            for (int u = g * PER; u < (g + 1) * PER; ++u)
                if (u < CA + CB) request_one(u);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    request(0, 0);
    request(BK < klast ? BK : klast, 1);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();                                               // waits for the requests, then for the waves
    operands(lds, 0, 0);
    int buf = 0;
    for (int k0 = 0; k0 < A.D; k0 += BK, buf ^= 1) {
        const char* const cur = lds + buf * BUF;
        const char* const nxt = lds + (buf ^ 1) * BUF;
        __builtin_amdgcn_sched_barrier(0);
        operands(cur, 1, 1);
        multiply(0);
        pattern();
        operands(cur, 2, 0);
        multiply(1);
        pattern();
        operands(cur, 3, 1);
        multiply(0);
        pattern();
        // A wave's own requests are counted by vmcnt; the barrier's fence does not wait for them (they are loads),
        // so the wait is written out: only then may the other waves read what this wave has requested.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();                                           // the next tile has arrived in every wave's part,
        // and this tile's buffer is free for the one after
        if constexpr (MB == 4) {
            request_from(k0 + 2 * BK < klast ? k0 + 2 * BK : klast, buf);
            last_slice(nxt);
        } else {
            request(k0 + 2 * BK < klast ? k0 + 2 * BK : klast, buf);
            operands(nxt, 0, 0);
            multiply(1);
            pattern();
        }
    }

    // Epilogue: bias, then the tile's half of the head (a tile never straddles V: V is a multiple of BN).  The
    // accumulators hold columns across lanes and rows across registers; stored as they are, an instruction would
    // write 128-byte pieces of two rows.  Each wave instead passes its block through LDS, 32 rows at a time (the
    // operand buffers are free by now), and writes whole row segments of 32 NB floats: 16 bytes per lane.  The staging
    // area is the wave's own, so nothing but the wave's own LDS operations is awaited, and all reads of 32 rows are under
    // way together (one wave per SIMD: read, wait and store in turn, with a barrier on either side, stood still for a
    // third of a launch of 20 k tiles).
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // the last (repeated) requests have landed
    __syncthreads();                                               // every wave has read its last operands
    constexpr int WCOLS = 32 * NB, SP = WCOLS + 4;                 // staging pitch in floats: rows 4 apart differ in bank
    float* const stage = reinterpret_cast<float*>(lds) + wave * 32 * SP;
    float* out = n0 < A.V ? A.centre : A.radius;
    const int cwave = (n0 < A.V ? n0 : n0 - A.V) + wn * WCOLS;     // first output column of the wave's block
    float bj[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) bj[j] = A.bias ? A.bias[n0 + wn * WCOLS + j * 32 + lrow] : 0.f;
    constexpr int LPR = WCOLS / 4, RPI = 64 / LPR, ST = 32 / RPI;  // lanes per row segment, rows per store instruction, stores
    const int srow = lane / LPR, scol = (lane % LPR) * 4;
    const bool whole = m0 + BM <= A.N;                             // uniform: no row of the tile past the end of the batch
    const int64_t row0 = m0 + wm * 32 * MB + srow;
    float* const orow = out + row0 * A.stride + cwave + scol;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                stage[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * SP + j * 32 + lrow] = acc[i][j][v] + bj[j];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        f32x4 val[ST];
#pragma unroll
        for (int t = 0; t < ST; ++t) val[t] = *reinterpret_cast<const f32x4*>(&stage[(t * RPI + srow) * SP + scol]);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int t = 0; t < ST; ++t)
            if (whole || row0 + i * 32 + t * RPI < A.N)
                *reinterpret_cast<f32x4*>(&orow[(int64_t)(i * 32 + t * RPI) * A.stride]) = val[t];
    }
}

template <int MB, int NB>
hipError_t launch_tile(const HeadArgs& a, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    constexpr int BM = 64 * MB, BN = 64 * NB;
    constexpr size_t lds_bytes = (size_t)2 * (BM + BN) * ROWB;                     // 64 KB or 128 KB of the 160 KB
    static_assert(lds_bytes <= 160 * 1024, "tile does not fit the LDS of a compute unit");
    if (lds_bytes > 64 * 1024) {
        // more than the default limit for dynamic LDS: raised for this kernel once per device (an attribute of the
        // function on the device that is current)
        static std::mutex mu;
        static bool raised[64] = {};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
        std::lock_guard<std::mutex> lock(mu);
        if (!raised[dev]) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&interhead_gemm_kernel<MB, NB>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
            if (e != hipSuccess) return e;
            raised[dev] = true;
        }
    }
    HeadArgs args = a;
    args.row_tiles = (int32_t)((a.N + BM - 1) / BM);
    args.col_tiles = 2 * a.V / BN;
    const unsigned grid = (unsigned)args.row_tiles * (unsigned)args.col_tiles;
    if (ev_start && ev_stop)
        hipExtLaunchKernelGGL((interhead_gemm_kernel<MB, NB>), dim3(grid), dim3(256), lds_bytes, stream, ev_start,
                              ev_stop, 0, args);
    else
        hipLaunchKernelGGL((interhead_gemm_kernel<MB, NB>), dim3(grid), dim3(256), lds_bytes, stream, args);
    return hipGetLastError();
}

// ---- many rows -------------------------------------------------------------------------------------------------------

// 256 x 128 workgroup tiles, 32 deep, four waves in a 2 x 2 grid of 128 x 64 (4 x 2 matrix blocks, 128 accumulator registers): two
// workgroups share a compute unit, so that one multiplies while the other waits at a barrier, starts a tile or writes one
// out.  For batches whose tiles have a compute unit each, and vocabularies that are not a multiple of 256; a large batch does better with the larger tile, which brings a third less into LDS per matrix instruction.
// Three stages of 24 KiB: a slice is requested two slices ahead and awaited by count (the one behind it may still be under
// way).  A tile row is four 16-byte chunks, chunk q of row r at position q ^ ((r / 4) % 4): four rows fill the 64 banks, and
// any 16 consecutive rows at the same k cover every bank once.
constexpr int BK2 = 32, ROWB2 = BK2 * 2;

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
void interhead_pair_kernel(const HeadArgs A)
{
    constexpr int MB = 4, NB = 2, BM = 64 * MB, BN = 64 * NB, STAGES = 3;
    constexpr int CA = BM / 64, CB = BN / 64, LOADS = CA + CB;     // load instructions per wave and slice (16 rows each)
    constexpr int STAGE = (BM + BN) * ROWB2;
    extern __shared__ __attribute__((aligned(1024))) char lds[];   // [STAGES][hidden tile, weight tile]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    // the tiles are dealt by XCD, see interhead_gemm_kernel
    int rt, ct;
    if (A.col_tiles % 8 == 0) {
        const int x = (int)(blockIdx.x & 7), local = (int)(blockIdx.x >> 3);
        rt = local % A.row_tiles;
        ct = (local / A.row_tiles) * 8 + x;
    } else {
        rt = (int)(blockIdx.x % A.row_tiles);
        ct = (int)(blockIdx.x / A.row_tiles);
    }
    const int64_t m0 = (int64_t)rt * BM;
    const int n0 = ct * BN;

    // Requests: instruction u of wave w covers the tile rows 16 (w + 4 u) .. + 15; lane l asks for row + l / 4 and, of that row,
    // the chunk that belongs at position l % 4.
    uint32_t oa[CA], ob[CB];
    const int rl = lane >> 2, chunk = (lane & 3) ^ ((rl >> 2) & 3);
    const int64_t last = A.N - 1 - m0;                             // >= 0: the tile starts inside the batch
#pragma unroll
    for (int u = 0; u < CA; ++u) {
        const int row = 16 * (wave + 4 * u) + rl;
        oa[u] = (uint32_t)(row <= last ? row : (int)last) * (uint32_t)A.D * 2u + (uint32_t)chunk * 16u;
    }
#pragma unroll
    for (int u = 0; u < CB; ++u) ob[u] = (uint32_t)(16 * (wave + 4 * u) + rl) * (uint32_t)A.D * 2u + (uint32_t)chunk * 16u;
    const gbytes baseA = (gbytes)(A.hidden + m0 * A.D), baseB = (gbytes)(A.weight + (int64_t)n0 * A.D);
    const int klast = A.D - BK2;                                   // (past the last slice the requests repeat it)
    uint64_t kA, kB;
    int dst;
    auto request_from = [&](int k0, int stage) {
        k0 = k0 < klast ? k0 : klast;
        kA = (uint64_t)baseA + (uint32_t)k0 * 2u;
        kB = (uint64_t)baseB + (uint32_t)k0 * 2u;
        dst = stage * STAGE + wave * 16 * ROWB2;
        asm volatile("" : "+s"(kA), "+s"(kB));
    };
    auto request_one = [&](int u) {
        if (u < CA) __builtin_amdgcn_global_load_lds((gptr)((gbytes)kA + oa[u < CA ? u : 0]), (lptr)(lds + dst + u * 64 * ROWB2), 16, 0, 0);
        else __builtin_amdgcn_global_load_lds((gptr)((gbytes)kB + ob[u < CA ? 0 : u - CA]),
                                              (lptr)(lds + dst + BM * ROWB2 + (u - CA) * 64 * ROWB2), 16, 0, 0);
    };

    f32x16 acc[MB][NB];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // Operand reads: lane l reads row l % 32 of each 32-row block; its chunk in step sl (k 16 sl .. + 15) is 2 sl + l / 32.
    const int lrow = lane & 31, sw = (lane >> 5) ^ ((lrow >> 2) & 3);
    const int offA = (wm * 32 * MB + lrow) * ROWB2, offB = BM * ROWB2 + (wn * 32 * NB + lrow) * ROWB2;
    bf16x8 a[2][MB], b[2][NB];
    auto operand = [&](int stage, int sl, int set, int q) {        // operand q of a step: the MB of A, then the NB of B
        const char* const tile = lds + stage * STAGE + ((2 * sl) ^ sw) * 16;
        if (q < MB) a[set][q < MB ? q : 0] = *reinterpret_cast<const bf16x8*>(tile + offA + q * 32 * ROWB2);
        else b[set][q < MB ? 0 : q - MB] = *reinterpret_cast<const bf16x8*>(tile + offB + (q - MB) * 32 * ROWB2);
    };
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        request_from(t * BK2, t);
#pragma unroll
        for (int u = 0; u < LOADS; ++u) request_one(u);
    }
    request_from(2 * BK2, 2);
#pragma unroll
    for (int u = 0; u < LOADS; ++u) request_one(u);
    asm volatile("s_waitcnt vmcnt(%0)" :: "n"(2 * LOADS) : "memory");
    lds_join();
#pragma unroll
    for (int q = 0; q < MB + NB; ++q) operand(0, 0, 0, q);
    int stage = 0;
    for (int k0 = 0; k0 < A.D; k0 += BK2) {
        const int next = stage + 1 == STAGES ? 0 : stage + 1;
        __builtin_amdgcn_sched_barrier(0);
        // first step: the second step's operands are read meanwhile
#pragma unroll
        for (int g = 0; g < MB * NB; ++g) {
            acc[g / NB][g % NB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[0][g / NB], b[0][g % NB], acc[g / NB][g % NB], 0, 0, 0);
            if (g < MB + NB) operand(stage, 1, 1, g);
            __builtin_amdgcn_sched_barrier(0);
        }
        // Every wave holds its last operands of this slice: its stage is free for the slice three on.  The next slice has landed
        // when all but the LOADS requests behind it have.
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"(LOADS) : "memory");
        lds_join();
        request_from(k0 + STAGES * BK2, stage);
#pragma unroll
        for (int g = 0; g < MB * NB; ++g) {
            acc[g / NB][g % NB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[1][g / NB], b[1][g % NB], acc[g / NB][g % NB], 0, 0, 0);
            if (g < MB + NB) operand(next, 0, 0, g);
            if (g < LOADS) request_one(g);
            __builtin_amdgcn_sched_barrier(0);
        }
        stage = next;
    }

    // Epilogue: as in interhead_gemm_kernel, 32 rows at a time through the wave's own part of LDS.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // the last (repeated) requests have landed
    lds_join();                                                    // every wave has read its last operands
    constexpr int WCOLS = 32 * NB, SP = WCOLS + 4;
    float* const staged = reinterpret_cast<float*>(lds) + wave * 32 * SP;
    float* out = n0 < A.V ? A.centre : A.radius;                   // (V is a multiple of 128: a tile never straddles it)
    const int cwave = (n0 < A.V ? n0 : n0 - A.V) + wn * WCOLS;
    float bj[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) bj[j] = A.bias ? A.bias[n0 + wn * WCOLS + j * 32 + lrow] : 0.f;
    constexpr int LPR = WCOLS / 4, RPI = 64 / LPR, ST = 32 / RPI;
    const int srow = lane / LPR, scol = (lane % LPR) * 4;
    const bool whole = m0 + BM <= A.N;                             // uniform
    const int64_t row0 = m0 + wm * 32 * MB + srow;
    float* const orow = out + row0 * A.stride + cwave + scol;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                staged[(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * SP + j * 32 + lrow] = acc[i][j][v] + bj[j];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        f32x4 val[ST];
#pragma unroll
        for (int t = 0; t < ST; ++t) val[t] = *reinterpret_cast<const f32x4*>(&staged[(t * RPI + srow) * SP + scol]);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int t = 0; t < ST; ++t)
            if (whole || row0 + i * 32 + t * RPI < A.N)
                *reinterpret_cast<f32x4*>(&orow[(int64_t)(i * 32 + t * RPI) * A.stride]) = val[t];
    }
}

hipError_t launch_pair(const HeadArgs& a, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    constexpr size_t lds_bytes = (size_t)3 * (256 + 128) * ROWB2;  // 72 KB: two workgroups per compute unit
    {
        static std::mutex mu;
        static bool raised[64] = {};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
        std::lock_guard<std::mutex> lock(mu);
        if (!raised[dev]) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&interhead_pair_kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
            if (e != hipSuccess) return e;
            raised[dev] = true;
        }
    }
    HeadArgs args = a;
    args.row_tiles = (int32_t)((a.N + 255) / 256);
    args.col_tiles = 2 * a.V / 128;
    const unsigned grid = (unsigned)args.row_tiles * (unsigned)args.col_tiles;
    if (ev_start && ev_stop)
        hipExtLaunchKernelGGL(interhead_pair_kernel, dim3(grid), dim3(256), lds_bytes, stream, ev_start, ev_stop, 0, args);
    else
        hipLaunchKernelGGL(interhead_pair_kernel, dim3(grid), dim3(256), lds_bytes, stream, args);
    return hipGetLastError();
}

// ---- few rows --------------------------------------------------------------------------------------------------------

// The same maps for at most 32 rows (a drafted window or two): bound by reading the weights once.  A wave multiplies 32 output
// columns by all rows, on its own: its 32 weight rows stream through a ring of stages in LDS that only this wave writes and
// reads (a stage is a 64-deep slice: 4 KiB of weights and the same slice of the hidden states, 1 KiB per eight rows), so that
// nothing but its own count of outstanding loads has to be awaited -- no barrier, and STAGES - 1 slices per wave, 96 to 120 KiB
// per compute unit, on their way all the time (the 128 x 128 tile waited for one 32 KiB tile after another: 18.3 us for
// 8 x 1280 x 2 * 16384, 84 MB of weights).  KS waves of a workgroup share the columns and divide the depth when the vocabulary alone
// would leave compute units without work; their blocks are added up in LDS in a fixed order.
// The weights are the A operand: a lane then holds four consecutive output columns of one row per register group, a 16-byte
// store.
template <int HB> constexpr int few_stages() { return HB == 1 ? 7 : HB == 2 ? 6 : 4; }   // HB = eight-row groups of hidden states

template <int HB, int KS>
__global__ __launch_bounds__(256) void interhead_few_kernel(const HeadArgs A)
{
    constexpr int STAGES = few_stages<HB>(), STAGE = 4096 + HB * 1024, LOADS = 4 + HB;
    extern __shared__ __attribute__((aligned(1024))) char lds[];   // [4 waves][STAGES][STAGE]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int part = wave % KS, n0 = ((int)blockIdx.x * (4 / KS) + wave / KS) * 32;       // slice of the depth; first output column
    char* const ring = lds + wave * STAGES * STAGE;

    // requests: as in interhead_gemm_kernel, an instruction fills eight tile rows of 64 bf16, chunk q of row r at position
    // q ^ ((r / 2) % 8)
    const int rl = lane >> 3;
    const uint32_t pitch = (uint32_t)A.D * 2u;
    uint32_t ow[4], oh[HB];
#pragma unroll
    for (int u = 0; u < 4; ++u) ow[u] = (uint32_t)(8 * u + rl) * pitch + (uint32_t)((lane & 7) ^ ((4 * (u & 1)) | (rl >> 1))) * 16u;
#pragma unroll
    for (int u = 0; u < HB; ++u) {
        const int row = 8 * u + rl, last = (int)A.N - 1;           // (rows past the end of the batch repeat the last row)
        oh[u] = (uint32_t)(row < last ? row : last) * pitch + (uint32_t)((lane & 7) ^ ((4 * (u & 1)) | (rl >> 1))) * 16u;
    }
    const char* const baseW = reinterpret_cast<const char*>(A.weight + (int64_t)n0 * A.D);
    const char* const baseH = reinterpret_cast<const char*>(A.hidden);
    const int tiles = A.D / BK, per = (tiles + KS - 1) / KS;       // 64-deep slices, and of this wave
    const int first = part * per, count = max(0, min(tiles, first + per) - first);
    // (past its last slice a wave requests that one again: the number of outstanding loads stays what the waits assume)
    auto request = [&](int t, int stage) {
        const int k0 = (first + min(t, max(count - 1, 0))) * BK * 2;
        const int at = min(k0, (tiles - 1) * BK * 2);
        char* const d = ring + stage * STAGE;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            __builtin_amdgcn_global_load_lds((gptr)(baseW + at + ow[u]), (lptr)(d + u * 1024), 16, 0, 0);
#pragma unroll
        for (int u = 0; u < HB; ++u)
            __builtin_amdgcn_global_load_lds((gptr)(baseH + at + oh[u]), (lptr)(d + 4096 + u * 1024), 16, 0, 0);
    };
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    const int lrow = lane & 31, sw = (lane >> 5) ^ ((lrow >> 1) & 7);
    const int hrow = lrow < 8 * HB ? lrow : 8 * HB - 1;            // (columns past the batch: any row, never stored)
    const int hsw = (lane >> 5) ^ ((hrow >> 1) & 7);
#pragma unroll
    for (int t = 0; t < STAGES - 1; ++t) request(t, t);
    int stage = 0;
    for (int t = 0; t < count; ++t) {
        // the oldest slice has landed; the one that was read last is free for the request
        asm volatile("s_waitcnt vmcnt(%0)" :: "n"((STAGES - 2) * LOADS) : "memory");
        const char* const d = ring + stage * STAGE;
        bf16x8 w[4], x[4];
#pragma unroll
        for (int sl = 0; sl < 4; ++sl) {
            w[sl] = *reinterpret_cast<const bf16x8*>(d + lrow * ROWB + ((2 * sl) ^ sw) * 16);
            x[sl] = *reinterpret_cast<const bf16x8*>(d + 4096 + hrow * ROWB + ((2 * sl) ^ hsw) * 16);
        }
        request(t + STAGES - 1, stage == 0 ? STAGES - 1 : stage - 1);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int sl = 0; sl < 4; ++sl) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[sl], x[sl], acc, 0, 0, 0);
        stage = stage + 1 == STAGES ? 0 : stage + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");                // the repeated requests have landed
    if constexpr (KS > 1) {
        // the other waves' blocks, [register][lane], added by the first of the KS waves in order
        float* const block = reinterpret_cast<float*>(ring);
        if (part > 0) {
#pragma unroll
            for (int v = 0; v < 16; ++v) block[v * 64 + lane] = acc[v];
        }
        __syncthreads();
        if (part > 0) return;
#pragma unroll
        for (int o = 1; o < KS; ++o) {
            const float* const other = reinterpret_cast<const float*>(ring + o * STAGES * STAGE);
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[v] += other[v * 64 + lane];
        }
    }
    if (lrow >= A.N) return;
    float* const out = n0 < A.V ? A.centre : A.radius;             // (V is a multiple of 128: a block never straddles it)
    const int col = (n0 < A.V ? n0 : n0 - A.V) + 4 * (lane >> 5);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        f32x4 val = {acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]};
        if (A.bias) {
            const float* const b = A.bias + n0 + 4 * (lane >> 5) + 8 * g;
            val += f32x4{b[0], b[1], b[2], b[3]};
        }
        *reinterpret_cast<f32x4*>(&out[(int64_t)lrow * A.stride + col + 8 * g]) = val;
    }
}

template <int HB, int KS>
hipError_t launch_few(const HeadArgs& a, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    constexpr size_t lds_bytes = (size_t)4 * few_stages<HB>() * (4096 + HB * 1024);       // 128 to 144 KB of the 160 KB
    {
        static std::mutex mu;
        static bool raised[64] = {};
        int dev = 0;
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
        std::lock_guard<std::mutex> lock(mu);
        if (!raised[dev]) {
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&interhead_few_kernel<HB, KS>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
            if (e != hipSuccess) return e;
            raised[dev] = true;
        }
    }
    const unsigned grid = (unsigned)(2 * a.V / 32 / (4 / KS));
    if (ev_start && ev_stop)
        hipExtLaunchKernelGGL((interhead_few_kernel<HB, KS>), dim3(grid), dim3(256), lds_bytes, stream, ev_start, ev_stop, 0, a);
    else
        hipLaunchKernelGGL((interhead_few_kernel<HB, KS>), dim3(grid), dim3(256), lds_bytes, stream, a);
    return hipGetLastError();
}
template <int HB>
hipError_t launch_few_split(const HeadArgs& a, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    // 2 V / 32 column blocks, a wave each: the depth is divided where they leave a compute unit less than three waves
    const int blocks = 2 * a.V / 32, wanted = 3 * compute_units();
    if (blocks >= wanted) return launch_few<HB, 1>(a, stream, ev_start, ev_stop);
    if (2 * blocks >= wanted) return launch_few<HB, 2>(a, stream, ev_start, ev_stop);
    return launch_few<HB, 4>(a, stream, ev_start, ev_stop);
}

}  // namespace

hipError_t launch_interhead(const HeadArgs& args, hipStream_t stream, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    if (args.N <= 0) return hipSuccess;
    static_assert(kHeadTileCols == 128, "the small tile is the one the C ABI's shape check is written for");
    if (args.N <= 8) return launch_few_split<1>(args, stream, ev_start, ev_stop);
    if (args.N <= 16) return launch_few_split<2>(args, stream, ev_start, ev_stop);
    if (args.N <= 32) return launch_few_split<4>(args, stream, ev_start, ev_stop);
    if (args.N <= 128) return launch_tile<2, 2>(args, stream, ev_start, ev_stop);
    // 256 x 256 tiles read the least per matrix instruction.  Where they are so few that 256 x 128 ones have a compute unit each,
    // those are as quick and twice as many (785 x 2240 x 2 * 2560: 51 -> 34.5 us, 512 x 1280 x 2 * 8192 51 -> 44, x 4096 98 -> 86);
    // two of them to a compute unit are slower than one large tile (512 rows, x 1280 x 2 * 10240 53.2 against 58.4, x 4096 101 /
    // 127, x 4096 x 2 * 14336 125 / 148).  An odd multiple of 128 has no large tiles: there, up to 256 rows, one round of
    // 128 x 128 (256 rows, x 4096 x 2 * 7296 57.4 against 66.7, x 4096 x 2 * 2176 50.5 / 60.9, x 1280 25.8 / 28.6, x 512 23.9 / 23.6),
    // or of half the compute units with it where the second row of tiles is half empty (160 rows, x 1280 x 2 * 7296 32.4 / 31.9,
    // x 3072 53.6 / 50.5, x 4096 x 2 * 2176 50.4 / 55.3).
    const int64_t cus = compute_units(), tiles = (args.N + 255) / 256 * (2 * (int64_t)args.V / 256);
    if (args.V % 256 == 0 && 2 * tiles > cus) return launch_tile<4, 4>(args, stream, ev_start, ev_stop);
    if (args.V % 256 != 0 && args.N <= 256 && 4 * (int64_t)args.V / 128 <= (args.N >= 192 ? cus : cus / 2)) return launch_tile<2, 2>(args, stream, ev_start, ev_stop);
    return launch_pair(args, stream, ev_start, ev_stop);
}

}  // namespace ciar

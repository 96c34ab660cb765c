// The dense transform of eq. (2) in fp32 matrix instructions, act(M H + X H0), for rows of any length up to 256: fp32 storage whose input width is no
// multiple of 4, and, where the caller asks for fp32 instructions (varco_set_matmul_terms), any. The instructions, their operands and their order are those
// of gemm_kernel in kernels_gemm.hip, so the bits are: a tile of 16 reduction steps is eight instructions, the t-th of which multiplies steps t and 8 + t,
// and the second tap follows in the same accumulators. Which of the two kernels takes a call depends on its number of rows (varco_gemm_rows_usable), and a
// row's result must not.
//
// A wavefront keeps 32 columns of the weights in registers, both taps', for all the rows that its workgroup walks over. Blocks of 32 rows come 16 lanes
// to a row, from any 4-byte address, one block ahead in registers, and lie in LDS as [tile][row][16 steps], the 16-byte pieces of every fourth row
// swapped so that fragments are read without a bank conflict. One LDS buffer, two barriers per block: the other workgroups of the compute unit
// multiply meanwhile. Bound by the matrix units (two taps of 233 steps -> 160, 211,211 rows: 51 % busy at 2.3 GHz with five of six wavefronts at work, 8 % vector
// instructions beside them, the rest waits, one wavefront to a SIMD; up to 256 steps two or three), in small launches by one block's chain. gemm_kernel's tiles of 128 rows x 128 columns in stages of 16 steps / this, us:
//   3,000 rows 218 -> 48 34.2 / 9.6, 130 -> 256 22.3 / 8.5, two taps 233 -> 160 59.9 / 16.5     20,000 rows two taps 55 -> 160 29.4 / 17.6
//   50,021 rows two taps 75 -> 200 64 / 50     200,000 rows 218 -> 160 264 / 186, 130 -> 256 192 / 154, two taps 233 -> 256 533 / 508, 55 -> 256 173 / 142
// and rows of aligned length: 3,000 rows 64 -> 128 12.0 / 6.1, 256 -> 256 29 / 11     50,021 rows 100 -> 256 45 / 33, two taps 128 -> 256 91 / 72
//   200,000 rows 128 -> 256 147 / 122, 256 -> 256 257 / 220     1,000,000 rows 100 -> 40 200 / 143, 256 -> 512 2,341 / 2,097
// (Blocks of 64 rows, two accumulators: fewer wavefronts, 50,021 rows 75; the next block's loads and LDS writes among the products, two buffers:
// two taps of 233 steps 490 instead of 508, two-wavefront workgroups lose by the LDS.)
#include <algorithm>
#include <type_traits>

#include "gemm_tile.h"
#include "varco_internal.h"

namespace {

constexpr int kRows = 32;            // rows of a block
constexpr int kColumns = 32;         // columns of a wavefront
constexpr int kTile = 16;            // reduction steps of a tile
constexpr int kPiece = 64;           // reduction steps of a row that 16 lanes fetch at a time
constexpr int kUnits = 256;          // compute units

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float any4 __attribute__((ext_vector_type(4), aligned(4)));

struct RowsGemm {
    const float* a[2];               // rows of the taps
    const float* b[2];               // their weights, k x n
    int64_t lda, ldb;
    int32_t m, n, k;
    float* c;
    int64_t ldc;
    int32_t accumulate, relu;
    int32_t groups, stride;          // groups of columns; workgroups of a group
};

// No load or store of this wavefront is on its way. Behind the products the next block has long arrived; if the compiler had to wait for it behind the
// stores of this one, whose number depends on the branch taken, it would wait for the stores as well.
constexpr int kLoaded = 0x0F70;

// Wavefronts that a SIMD holds: weights take 32 registers per 64 steps.
constexpr int resident(int pieces) { return pieces <= 2 ? 3 : pieces <= 4 ? 2 : 1; }

// J: 64-step pieces of a tap's row; WAVES: wavefronts, 32 columns each.
template <int J, int TAPS, int WAVES>
__global__ __launch_bounds__(64 * WAVES, resident(J * TAPS)) void rows_kernel(RowsGemm g) {
    constexpr int TILES = J * kPiece / kTile, RI = kRows / (4 * WAVES), PIECES = TAPS * RI * J;
    __shared__ __attribute__((aligned(16))) float smem[TAPS * TILES * kTile * kRows];
    const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, l32 = lane & 31, lk = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // the groups of one range of rows follow one another on one XCD: the rows come into a single L2
    const int32_t xcd = blockIdx.x & 7, within = blockIdx.x >> 3;
    const int32_t first = (within / g.groups) * 8 + xcd, n_blocks = (g.m + kRows - 1) / kRows, whole = g.m / kRows;
    if (first >= n_blocks || first >= g.stride) return;         // whole workgroup
    const int32_t n0 = ((within % g.groups) * WAVES + (wave + first) % WAVES) * kColumns;       // (a wavefront without columns: on every SIMD in turn)
    const bool mine = n0 < g.n;

    // weights: lane (column l32, half lk) holds steps 16 t + 8 lk + s
    float w[TAPS][TILES][8];
#pragma unroll
    for (int tap = 0; tap < TAPS; ++tap) {
        const uint32_t column = uint32_t(min(n0 + l32, g.n - 1));
#pragma unroll
        for (int t = 0; t < TILES; ++t)
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int32_t k = kTile * t + 8 * lk + s;
                w[tap][t][s] = load_at<float>(g.b[tap], 4u * (uint32_t(min(k, g.k - 1)) * uint32_t(g.ldb) + column));
            }
    }
#pragma unroll
    for (int tap = 0; tap < TAPS; ++tap)
#pragma unroll
        for (int t = TILES - 4; t < TILES; ++t)
#pragma unroll
            for (int s = 0; s < 8; ++s) w[tap][t][s] = kTile * t + 8 * lk + s < g.k ? w[tap][t][s] : 0.f;

    // this lane's rows and columns of a block; the piece that crosses the end of its row comes from four steps before the end
    const int row0 = wave * (4 * RI) + (lane >> 4);
    const uint32_t pitch = uint32_t(g.lda) * 4u;
    const int32_t last = kPiece * (J - 1) + 4 * l16;
    const uint32_t off = 16u * uint32_t(l16), off_last = 4u * uint32_t(min(last, g.k - 4));
    floatx4 x[TAPS * RI * J];
    auto fetch = [&](int32_t block, int p) __attribute__((always_inline)) {       // piece p of the block
        const int tap = p / (RI * J), i = p / J % RI, j = p % J;
        const int32_t b = min(block, n_blocks - 1), most = g.m - 1 - b * kRows;
        const char* const base = reinterpret_cast<const char*>(g.a[tap] + int64_t(b) * kRows * g.lda);
        x[p] = *reinterpret_cast<const any4*>(base + (uint32_t(min(row0 + 4 * i, most)) * pitch + (j + 1 < J ? off + 256u * j : off_last)));
    };
    // (that piece moves up by what it came early, by two steps and by one)
    const int32_t early = last < g.k ? max(last + 4 - g.k, 0) : 0;
    const bool two = early & 2, one = early & 1, beyond = last >= g.k;
    const int to = (l16 >> 2) * (kTile * kRows) + row0 * kTile;
    auto stash = [&](int p) __attribute__((always_inline)) {
        const int tap = p / (RI * J), i = p / J % RI, j = p % J;
        floatx4 v = x[p];
        if (j + 1 == J) {
            v = floatx4{two ? v[2] : v[0], two ? v[3] : v[1], two ? 0.f : v[2], two ? 0.f : v[3]};
            v = floatx4{one ? v[1] : v[0], one ? v[2] : v[1], one ? v[3] : v[2], one ? 0.f : v[3]};
            v = floatx4{beyond ? 0.f : v[0], beyond ? 0.f : v[1], beyond ? 0.f : v[2], beyond ? 0.f : v[3]};
        }
        *reinterpret_cast<floatx4*>(smem + to + ((tap * TILES + 4 * j) * kRows + 4 * i) * kTile + 4 * ((l16 & 3) ^ ((row0 >> 2) + i & 3))) = v;
    };

    const int swap = l32 >> 2 & 3;
#pragma unroll
    for (int p = 0; p < PIECES; ++p) fetch(first, p);
    __builtin_amdgcn_s_waitcnt(kLoaded);
    for (int32_t block = first; block < n_blocks; block += g.stride) {
#pragma unroll
        for (int p = 0; p < PIECES; ++p) stash(p);
#pragma unroll
        for (int p = 0; p < PIECES; ++p) fetch(block + g.stride, p);
        __syncthreads();
        floatx16 acc;
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[v] = 0.f;
        if (mine) {
            // half tiles, four steps of a lane, read two ahead of their products
            const float* const from = smem + l32 * kTile;
            constexpr int HALVES = TAPS * TILES * 2;
            floatx4 f[3];
            auto read = [&](int q) __attribute__((always_inline)) {
                return *reinterpret_cast<const floatx4*>(from + q / 2 * (kRows * kTile) + 4 * ((2 * lk + (q & 1)) ^ swap));
            };
            f[0] = read(0), f[1] = read(1);
#pragma unroll
            for (int q = 0; q < HALVES; ++q) {
                const int tap = q / (2 * TILES), t = q / 2 % TILES, s0 = 4 * (q & 1);
                if (q + 2 < HALVES) f[(q + 2) % 3] = read(q + 2);
                __builtin_amdgcn_sched_barrier(0);
                // the last tile: with s steps left, instructions from the s-th on would add zeros
                const int32_t left = t >= TILES - 4 ? g.k - kTile * t - s0 : kTile;
                if (left <= 0) continue;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    if (t >= TILES - 4 && s0 == 0 && s > 0 && s >= left) break;
                    acc = __builtin_amdgcn_mfma_f32_32x32x2f32(w[tap][t][s0 + s], f[q % 3][s], acc, 0, 0, 0);
                }
            }

        }
        __builtin_amdgcn_s_waitcnt(kLoaded);
        if (mine) {
            // a lane holds a row's columns 8 q + 4 lk .. + 3
            float* const c = g.c + (int64_t(block) * kRows + l32) * g.ldc + n0 + 4 * lk;
            auto put4 = [&](float* dst, floatx4 o) __attribute__((always_inline)) {
                o += g.accumulate ? floatx4(*reinterpret_cast<const any4*>(dst)) : floatx4{0.f, 0.f, 0.f, 0.f};
                if (g.relu) o = floatx4{fmaxf(o[0], 0.f), fmaxf(o[1], 0.f), fmaxf(o[2], 0.f), fmaxf(o[3], 0.f)};
                *reinterpret_cast<any4*>(dst) = o;
            };
            const bool inside = block < whole && n0 + kColumns <= g.n;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const floatx4 o = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
                float* const dst = c + 8 * q;
                const int32_t left = g.n - (n0 + 8 * q + 4 * lk);       // columns from this lane's first one on
                if (inside) {
                    put4(dst, o);
                } else if (block < whole || l32 < g.m - whole * kRows) {
                    // (element by element only what is left of a row: 500,009 rows 31 -> 30 36 us instead of 56, 17 -> 63 43 / 67)
                    if (left >= 4) {
                        put4(dst, o);
                    } else {
#pragma unroll
                        for (int v = 0; v < 3; ++v)
                            if (v < left) {
                                const float s = o[v] + (g.accumulate ? dst[v] : 0.f);
                                dst[v] = g.relu ? fmaxf(s, 0.f) : s;
                            }
                    }
                }
            }
        }
        __syncthreads();
    }
}

// Wavefronts of a workgroup: two where four would leave more of them without columns (200,000 rows 218 -> 48 110 with four, 71 with two, 130 -> 160 140 / 119;
// 130 -> 256 154 / 179).
int waves_of(int32_t n) {
    const int32_t units = (n + kColumns - 1) / kColumns;
    return (units + 3) / 4 * 4 > (units + 1) / 2 * 2 ? 2 : 4;
}

}  // namespace

bool varco_gemm_rows_usable(const GemmArgs& ga) {
    if (ga.m <= 0 || ga.n <= 0 || ga.k < 4 || ga.k > 256) return false;
    if (ga.a.dtype != VARCO_F32 || ga.b.dtype != VARCO_F32 || ga.c_dtype != VARCO_F32 || ga.a.transposed || ga.b.transposed) return false;
    if (ga.a.gate || ga.b.gate || ga.c_dual || ga.split_k > 1) return false;
    // offsets of a lane in 32 bits
    if (ga.a.ld > (int64_t(1) << 24) || ga.b.ld > (int64_t(1) << 21) || ga.a.ld < ga.k) return false;
    if (ga.k2 > 0 && (ga.k2 != ga.k || ga.a2.ld != ga.a.ld || ga.b2.ld != ga.b.ld || ga.a2.dtype != VARCO_F32 || ga.b2.dtype != VARCO_F32 || ga.a2.transposed ||
                      ga.b2.transposed || ga.a2.gate || ga.b2.gate))
        return false;
    // Where the tiles of gemm_kernel are ahead (us, there / here; rows of aligned length come here with fp32 instructions on request only):
    // few steps, once rows and results are more than the 256 MiB that the last cache holds: 1,000,000 rows 31 -> 47 98 / 119, 1,250,003 rows 15 -> 44
    // 97 / 114, 17 -> 47 121 / 142, two taps 16 -> 64 92 / 126, but 1,000,000 rows 17 -> 44 84 / 56, 33 -> 47 126 / 115, and 700,001 rows 31 -> 47 67 / 57;
    // results that no cache holds: 1,000,000 rows 17 -> 256 305 / 387, 33 -> 256 389 / 399, but 63 -> 256 495 / 410 and 200,000 rows 17 -> 256 64 / 48
    const bool two = ga.k2 > 0, aligned = ga.k % 4 == 0 && ga.a.ld % 4 == 0 && (reinterpret_cast<uintptr_t>(ga.a.ptr) & 15u) == 0;
    const int64_t out = int64_t(ga.m) * ga.n * 4, bytes = out + int64_t(ga.m) * ga.k * (two ? 8 : 4);
    if (ga.k <= (two ? 16 : 32) && bytes > (int64_t(256) << 20)) return false;
    if (!two && ga.k <= 48 && out > (int64_t(240) << 20)) return false;
    // few steps and rows fetched by four groups: 100,003 rows 17 -> 512 61 / 66 (aligned 16 -> 512 46 / 67), but 384 50 / 35 and 50,021 rows 512 36 / 32
    if (!two && ga.k <= 32 && ga.n > 384 && (aligned || ga.m > 64'000)) return false;
    // one wavefront to a SIMD and four of them to a workgroup: two taps 200,000 rows 233 -> 384 747 / 779, 512 950 / 959, but 320 735 / 647 and 20,000
    // rows 384 103 / 91; 1,000,003 rows 255 -> 200 2,354 / 2,450, 211 -> 256 2,073 / 2,140, but 193 -> 256 1,990 / 1,970 and 700,001 rows level; aligned
    // ones earlier, 204 -> 200 1,846 / 2,045, 128 1,016 / 1,090, 200,003 rows 224 -> 256 477 / 495, but 192 -> 256 415 / 401
    const int32_t pieces = (ga.k + kPiece - 1) / kPiece * (two ? 2 : 1);
    if (pieces <= 4 || waves_of(ga.n) == 2) return true;
    if (ga.n > 256 && ga.m >= 100'000) return false;
    return !(ga.n > (aligned ? 64 : 128) && ga.k > (aligned ? 192 : 208) && ga.m > (aligned ? 150'000 : 800'000));
}

hipError_t varco_launch_gemm_rows(const GemmArgs& ga, hipStream_t stream, const LaunchTag& tag) {
    RowsGemm g{};
    g.a[0] = static_cast<const float*>(ga.a.ptr), g.a[1] = static_cast<const float*>(ga.a2.ptr);
    g.b[0] = static_cast<const float*>(ga.b.ptr), g.b[1] = static_cast<const float*>(ga.b2.ptr);
    g.lda = ga.a.ld, g.ldb = ga.b.ld;
    g.m = ga.m, g.n = ga.n, g.k = ga.k;
    g.c = static_cast<float*>(ga.c), g.ldc = ga.ldc;
    g.accumulate = ga.accumulate ? 1 : 0, g.relu = ga.relu ? 1 : 0;
    const int waves = waves_of(ga.n), taps = ga.k2 > 0 ? 2 : 1, pieces = (ga.k + kPiece - 1) / kPiece;
    const int32_t n_blocks = (ga.m + kRows - 1) / kRows, columns = waves * kColumns;
    g.groups = (ga.n + columns - 1) / columns;
    g.stride = std::max(8, kUnits * 4 * resident(pieces * taps) / waves / g.groups / 8 * 8);
    const dim3 grid{unsigned((std::min(g.stride, n_blocks) + 7) / 8 * 8 * g.groups)};
    tag.begin(stream);
    using std::integral_constant;
    auto go = [&](auto j, auto t) {
        constexpr int J = decltype(j)::value, TAPS = decltype(t)::value;
        if (waves == 2)
            hipLaunchKernelGGL((rows_kernel<J, TAPS, 2>), grid, dim3(128), 0, stream, g);
        else
            hipLaunchKernelGGL((rows_kernel<J, TAPS, 4>), grid, dim3(256), 0, stream, g);
    };
    auto with_taps = [&](auto j) {
        if (taps == 2)
            go(j, integral_constant<int, 2>{});
        else
            go(j, integral_constant<int, 1>{});
    };
    switch (pieces) {
        case 1: with_taps(integral_constant<int, 1>{}); break;
        case 2: with_taps(integral_constant<int, 2>{}); break;
        case 3: with_taps(integral_constant<int, 3>{}); break;
        default: with_taps(integral_constant<int, 4>{});
    }
    tag.end(stream);
    return hipGetLastError();
}

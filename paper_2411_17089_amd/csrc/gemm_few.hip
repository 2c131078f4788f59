// Token GEMM for gfx950 and at most 8 rows: y[M, N] = x[M, K] . W[N, K]^T + bias (decode with few sequences).
//
// With so few rows the product is a read of W and nothing else, so the kernel is laid out for the read: the rate to reach is
// that of a plain loop of non-temporal 16-byte loads (6.4 - 6.9 TB/s over 100 - 400 MB here), against which the kernels for
// up to 64 rows, which take W through LDS or in the operand layout of the 16 x 16 MFMA, reach 4.7 - 5.7.
//   - v_mfma_f32_4x4x4_16b_f16: 16 independent products of 4 W rows by 4 tokens over 4 columns of K.  A lane owns 16 bytes
//     of one W row, so a wave load covers 4 rows x 256 contiguous bytes and goes straight into operand registers: no LDS, no
//     barrier, no transposition, and 4 tokens waste nothing where a 16 x 16 tile would waste three quarters.
//   - x stays in registers: the 8 waves of a workgroup cut K among themselves, a wave holds its part of x (M x K / 8) and
//     streams W rows past it, four at a time, the next four in flight.  Read again for every few rows, x cost as many
//     requests as W (M = 3, W of 5120 x 20480: 40 us that way, 33 with x in registers, 38 with the kernel for 64 rows).
//   - one workgroup per compute unit, each with an even share of the rows, strided by the grid so that the workgroups read
//     neighbouring rows at any time; twice or three times as many are up to 4 % slower with 3 tokens or more.
//   - the 16 partial products are folded over the lanes as they come (8 instructions for 4 rows x 4 tokens); the eight waves
//     meet in LDS once, at the end, behind the only barrier.
//   - where K / 8 is more than a wave can hold (P pieces of 128), W is walked in S column segments, the sums of a segment
//     are added to the wave's own in LDS.
// us per launch over rotating weights, the kernels for 64 rows -> this one, M = 1 / 4 / 8:
//   4096 x 4096    9.8 ->  7.3,  9.8 ->  7.6,  9.8 ->  8.1       12288 x 4096  21.5 -> 16.8, 21.5 -> 17.0, 21.6 -> 17.7
//   16384 x 4096  26.0 -> 21.6, 25.8 -> 21.8, 25.8 -> 22.5       4096 x 16384  27.4 -> 23.2, 27.4 -> 24.1, 27.5 -> 27.4
//   50272 x 4096  72.2 -> 61.6, 72.9 -> 62.1, 75.2 -> 64.1       22016 x 4096  33.7 -> 28.4, 33.8 -> 28.7, 33.9 -> 29.6
//   7168 x 7168   21.1 -> 17.6, 21.2 -> 18.1, 21.2 -> 18.7       7168 x 28672  72.5 -> 60.8, 72.8 -> 62.7, 72.9 -> 66.2
#include "gemm_few.h"
#include "silu.h"

#include <algorithm>
#include <type_traits>

namespace kvpr {
namespace {

typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef _Float16 half4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int PIECE = 128;       // columns of K that a wave load covers

template <int CTRL>
__device__ __forceinline__ float rotate_row(float v) {   // within 16 lanes
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xf, 0xf, true));
}
// lanes 0 .. 31 get the sum of a over the two halves of the wave, lanes 32 .. 63 that of b
__device__ __forceinline__ float fold32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_int(a), __float_as_int(b), false, false);
    return __int_as_float(r[0]) + __int_as_float(r[1]);
}
// as fold32 for the two rows of 16 lanes in each half
__device__ __forceinline__ float fold16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_int(a), __float_as_int(b), false, false);
    return __int_as_float(r[0]) + __int_as_float(r[1]);
}

// MQ: tokens in fours.  P: pieces of K that a wave holds at a time (every wave has P or P - 1 of them in every segment).
// A unit is 4 output features, or 2 x 4: the gate and the up rows of 4 features of a gated FFN, or 4 features of a head and
// their rotary partners.
// NORM: the rows of x are normalised in registers, where all of them are (one segment), while the first rows of W are on
// their way.  A norm of its own was a launch of 4.5 us with a round trip through memory in front of each of a layer's two
// wide products, the rotation one of 5 us behind the first (one token through 4 layers of hidden 4096, batch 1: 692 -> 658 us; 3
// rotary layers, batch 3: 504 -> 482).
// What comes with the product: nothing, the norm, or copies by extra workgroups (each an instantiation of its own: looking for
// copies costs a launch of 7 us 0.2).
enum class FewExtra { none, norm, copies };

// AGAIN: ordinary loads of W instead of non-temporal ones, for weights that the next kernels read again.  From memory the
// non-temporal ones are the faster (12288 x 4096, M = 1: 17.7 us against 18.6, 7168 x 28672: 64 against 71), but they leave nothing
// behind in the Infinity Cache.  In a single-layer call the recomputation reads [Wk; Wv] right after the projection has, and with few
// rows that read is what it takes.  6 layers called in turn, 24 positions, split 10, non-temporal / ordinary (kernels for up to 64
// rows): hidden 4096, batch 1 60.0 / 56.7 us (78.7), hidden 5120, batch 4 97.4 / 87.8 (104.2), hidden 7168, batch 6 166 / 155 (159);
// no recomputation: hidden 5120, batch 1 47.6 / 49.5, hidden 7168, batch 1 78 / 82.
template <int MQ, int P, FewForm FORM, int WAVES, FewExtra EXTRA, bool AGAIN = false>
__global__ __launch_bounds__(WAVES * 64) void few_tokens(const FewTokens a, int units, int segments, int grid, const CopyJob beside) {
    // rows four at a time: enough of them that a wave has at least four loads in flight behind the ones it works on
    constexpr int R = P == 1 ? 4 : P == 2 ? 2 : 1;
    constexpr int PER_UNIT = FORM == FewForm::plain ? 1 : 2;
    constexpr bool NORM = EXTRA == FewExtra::norm;
    if constexpr (EXTRA == FewExtra::copies)
        if ((int)blockIdx.x >= grid) {
            run_copy_job(beside, blockIdx.x - grid);
            return;
        }
    extern __shared__ float red[];                            // [group of 4 rows][quad of tokens][row][token][wave]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r4 = lane & 3, chunk = lane >> 2;
    const int groups = (units - (int)blockIdx.x + grid - 1) / grid * PER_UNIT;
    const int steps = (groups + R - 1) / R;
    auto row_of = [&](int g) {                                // first W row of this workgroup's group g
        const int unit = blockIdx.x + g / PER_UNIT * grid;
        if constexpr (FORM == FewForm::gated) return unit * 4 + (g & 1) * (a.N / 2);
        if constexpr (FORM == FewForm::rotary) {
            const int per_head = a.head_dim / 8;
            return unit / per_head * a.head_dim + unit % per_head * 4 + (g & 1) * (a.head_dim / 2);
        }
        return unit * 4;
    };
    __shared__ float stats[2][WAVES][MQ * 4];                 // sums over a wave's columns, then of squared deviations
    const int pieces = a.K / PIECE, run0 = pieces * wave / WAVES, run = pieces * (wave + 1) / WAVES - run0;

    for (int s = 0; s < segments; ++s) {
        const int p0 = run0 + run * s / segments, len = run0 + run * (s + 1) / segments - p0;
        const int k0 = p0 * PIECE + chunk * 8;
        auto walk = [&](auto count) {
            constexpr int CNT = decltype(count)::value;
            if constexpr (CNT == 0) {                         // fewer pieces than waves: K < 1024
                if constexpr (NORM) {
                    if (lane < MQ * 4) stats[0][wave][lane] = stats[1][wave][lane] = 0.f;
                    if (a.norm == 1) __syncthreads();
                    __syncthreads();
                }
                for (int i = lane; i < groups * MQ * 16; i += 64) red[i * WAVES + wave] = 0.f;
            } else {
                half8 xf[MQ][CNT];
#pragma unroll
                for (int q = 0; q < MQ; ++q)
#pragma unroll
                    for (int u = 0; u < CNT; ++u)
                        xf[q][u] = *reinterpret_cast<const half8*>(a.x + (int64_t)min(q * 4 + r4, a.M - 1) * a.K + k0 + u * PIECE);
                half8 gv[NORM ? CNT : 1], bv[NORM ? CNT : 1];
                if constexpr (NORM) {
#pragma unroll
                    for (int u = 0; u < CNT; ++u) {
                        gv[u] = *reinterpret_cast<const half8*>(a.norm_g + k0 + u * PIECE);
                        bv[u] = a.norm == 1 ? *reinterpret_cast<const half8*>(a.norm_b + k0 + u * PIECE) : half8{};
                    }
                }
                struct Rows { half8 w[R][CNT]; };
                auto load = [&](Rows& f, int st) {            // beyond the last group or row: the last one again, not stored
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        const _Float16* p = a.W + (int64_t)min(row_of(min(st * R + r, groups - 1)) + r4, a.N - 1) * a.K + k0;
#pragma unroll
                        for (int u = 0; u < CNT; ++u) {
                            const half8* from = reinterpret_cast<const half8*>(p + u * PIECE);
                            f.w[r][u] = AGAIN ? *from : __builtin_nontemporal_load(from);
                        }
                    }
                };
                auto multiply = [&](const Rows& f, int st) {
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        floatx4 acc[MQ];
#pragma unroll
                        for (int q = 0; q < MQ; ++q) acc[q] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int u = 0; u < CNT; ++u)
#pragma unroll
                            for (int q = 0; q < MQ; ++q) {
                                const half8 w = f.w[r][u], x = xf[q][u];
                                acc[q] = __builtin_amdgcn_mfma_f32_4x4x4f16(half4{w[0], w[1], w[2], w[3]}, half4{x[0], x[1], x[2], x[3]}, acc[q], 0, 0, 0);
                                acc[q] = __builtin_amdgcn_mfma_f32_4x4x4f16(half4{w[4], w[5], w[6], w[7]}, half4{x[4], x[5], x[6], x[7]}, acc[q], 0, 0, 0);
                            }
                        const int g = st * R + r;
                        // element e of a lane is W row e by token lane % 4, over the columns of its chunk: summed over the
                        // chunks, row e ends up in the 16 lanes from 16 e
#pragma unroll
                        for (int q = 0; q < MQ; ++q) {
                            float v = fold16(fold32(acc[q][0], acc[q][2]), fold32(acc[q][1], acc[q][3]));
                            v += rotate_row<0x124>(v);        // row_ror:4
                            v += rotate_row<0x128>(v);        // row_ror:8
                            if ((lane & 15) < 4 && g < groups) {
                                float* at = red + ((g * MQ + q) * 16 + (lane >> 4) * 4 + r4) * WAVES + wave;
                                *at = s == 0 ? v : *at + v;
                            }
                        }
                    }
                };
                // two groups of rows are on their way at any time; with a norm both from the start, since it takes as long as the
                // first two take to be read (with one the product of 12288 x 4096 took 20 us behind it, with two 18.5)
                Rows f0, f1;
                load(f0, 0);
                if constexpr (NORM) load(f1, 1);
                if constexpr (NORM) {
                    __builtin_amdgcn_sched_barrier(0);
                    // Float copies of x kept from one pass over it to the next would be 8 registers a piece, 112 with 7 pieces of 8
                    // tokens, and up to 67 of the 256 went to scratch (12 kernels, hidden 6144 and more).  Converted anew in
                    // each pass nothing does: token through 2 layers of hidden 7168, M = 1 / 4 / 8: 582 / 647 / 810 -> 561 / 615
                    // / 729 us (norm as a launch of its own 592 / 622 / 729); hidden 4096 and 5120 as before.
                    auto forget = [&]() {
#pragma unroll
                        for (int q = 0; q < MQ; ++q)
#pragma unroll
                            for (int u = 0; u < CNT; ++u) asm volatile("" : "+v"(xf[q][u]));
                    };
                    // f(token quad, element) summed over a token's row
                    auto row_sum = [&](int pass, float (&out)[MQ], auto&& f) {
                        forget();
#pragma unroll
                        for (int q = 0; q < MQ; ++q) {
                            float v = 0.f;
#pragma unroll
                            for (int u = 0; u < CNT; ++u)
#pragma unroll
                                for (int e = 0; e < 8; ++e) v += f(q, (float)xf[q][u][e]);
                            v += rotate_row<0x124>(v);
                            v += rotate_row<0x128>(v);
                            v += __shfl_xor(v, 16);
                            v += __shfl_xor(v, 32);
                            if (lane < 4) stats[pass][wave][q * 4 + lane] = v;
                        }
                        __syncthreads();
#pragma unroll
                        for (int q = 0; q < MQ; ++q) {
                            out[q] = 0.f;
#pragma unroll
                            for (int w = 0; w < WAVES; ++w) out[q] += stats[pass][w][q * 4 + r4];
                        }
                    };
                    float mean[MQ], var[MQ];
#pragma unroll
                    for (int q = 0; q < MQ; ++q) mean[q] = 0.f;
                    if (a.norm == 1) {
                        row_sum(0, mean, [](int, float v) { return v; });
#pragma unroll
                        for (int q = 0; q < MQ; ++q) mean[q] /= a.K;
                    }
                    row_sum(1, var, [&](int q, float v) { return (v - mean[q]) * (v - mean[q]); });
                    forget();
#pragma unroll
                    for (int q = 0; q < MQ; ++q) {
                        const float rstd = rsqrtf(var[q] / a.K + 1e-5f);
#pragma unroll
                        for (int u = 0; u < CNT; ++u) {
#pragma unroll
                            for (int e = 0; e < 8; ++e) {
                                const float t = ((float)xf[q][u][e] - mean[q]) * rstd * (float)gv[u][e];
                                xf[q][u][e] = (_Float16)(a.norm == 1 ? t + (float)bv[u][e] : t);
                            }
                            if (a.xn && blockIdx.x == 0 && q * 4 + r4 < a.M)
                                *reinterpret_cast<half8*>(a.xn + (int64_t)(q * 4 + r4) * a.K + k0 + u * PIECE) = xf[q][u];
                        }
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
                int st = 0;
                if constexpr (NORM) {
                    for (; st + 3 < steps; st += 2) {
                        multiply(f0, st);
                        __builtin_amdgcn_sched_barrier(0);
                        load(f0, st + 2);
                        __builtin_amdgcn_sched_barrier(0);
                        multiply(f1, st + 1);
                        __builtin_amdgcn_sched_barrier(0);
                        load(f1, st + 3);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    multiply(f0, st);
                    if (st + 2 < steps) {
                        __builtin_amdgcn_sched_barrier(0);
                        load(f0, st + 2);
                        __builtin_amdgcn_sched_barrier(0);
                        multiply(f1, st + 1);
                        multiply(f0, st + 2);
                    } else if (st + 1 < steps) {
                        multiply(f1, st + 1);
                    }
                    return;
                }
                for (; st + 2 < steps; st += 2) {
                    load(f1, st + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(f0, st);
                    __builtin_amdgcn_sched_barrier(0);
                    load(f0, st + 2);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(f1, st + 1);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (st + 1 < steps) {
                    load(f1, st + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(f0, st);
                    multiply(f1, st + 1);
                } else {
                    multiply(f0, st);
                }
            }
        };
        // two loops, so that the number of loads behind the ones that are waited for is known
        if (len == P) walk(std::integral_constant<int, P>{});
        else walk(std::integral_constant<int, P - 1>{});
    }
    __syncthreads();

    auto sum = [&](int i) {                                   // over the waves
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < WAVES; w += 4) {
            const float4 f = *reinterpret_cast<const float4*>(red + i * WAVES + w);
            v += (f.x + f.y) + (f.z + f.w);
        }
        return v;
    };
    for (int t = threadIdx.x; t < groups / PER_UNIT * MQ * 16; t += WAVES * 64) {
        const int m = (t >> 4) % MQ * 4 + (t & 3), unit = (t >> 4) / MQ, i = t & 15;
        const int n = row_of(unit * PER_UNIT) + (i >> 2);
        if (m >= a.M) continue;
        const int at = (unit * PER_UNIT * MQ + (t >> 4) % MQ) * 16 + i;
        if constexpr (FORM == FewForm::rotary) {
            const int h = a.N / 3, n2 = n + a.head_dim / 2;
            float v1 = sum(at), v2 = sum(at + MQ * 16);
            if (a.bias) {
                v1 += (float)a.bias[n];
                v2 += (float)a.bias[n2];
            }
            if (n < 2 * h) {
                const float2 cs = a.rope[n % a.head_dim];
                const float r1 = v1 * cs.x - v2 * cs.y, r2 = v2 * cs.x + v1 * cs.y;
                v1 = r1;
                v2 = r2;
            }
            if (n < h) {
                a.y32[(int64_t)m * h + n] = v1;
                a.y32[(int64_t)m * h + n2] = v2;
            } else {
                a.y16[(int64_t)m * a.ld16 + n - h] = (_Float16)v1;
                a.y16[(int64_t)m * a.ld16 + n2 - h] = (_Float16)v2;
            }
        } else if constexpr (FORM == FewForm::gated) {
            // both rounded to float16, as a product stored in between would have them
            const float gate = (float)(_Float16)sum(at), up = (float)(_Float16)sum(at + MQ * 16);
            a.y16[(int64_t)m * a.ld16 + n] = (_Float16)silu_mul(gate, up);
        } else {
            if (n >= a.N) continue;
            float v = sum(at);
            if (a.bias) v += (float)a.bias[n];
            if (a.relu) v = fmaxf(v, 0.f);
            if (n < a.out_f32_cols) {
                a.y32[(int64_t)m * a.out_f32_cols + n] = v;
            } else {
                // with a residual: rounded once by itself and once more with the residual added
                const int64_t to = (int64_t)m * a.ld16 + (n - a.out_f32_cols);
                _Float16 o = (_Float16)v;
                if (a.res) o = (_Float16)((float)o + (float)a.res[to]);
                a.y16[to] = o;
            }
        }
    }
}

// How a product is cut: waves and the pieces of K that each holds at a time, column segments, workgroups, bytes of LDS for the sums
// of one of them.
struct FewPlan {
    int waves, pieces, segments, grid, lds;
};

// Waves and pieces.  A wave has 128 registers for its part of x and for two groups of rows: 8 pieces with up to 4 tokens,
// 7 with up to 8.  One segment where that is enough (K = 7168, M = 8: 18.5 us against 18.9 in two), else with more than 4
// tokens segments of at most 4 pieces, whose rows are fewer registers to wait for at the end of one (K = 11008: 18.9 against
// 19.3 us, K = 20480: 37.1 against 38.0).  Where K is a multiple of 16384 the runs of 8 waves are multiples of 4 KiB apart and
// crowd the same channels: 4 waves, of 7 pieces at a time (4096 x 16384, M = 1 / 3 / 8: 24.7 / 25.7 / 29.3 -> 23.3 / 23.3 / 27.1
// us; elsewhere they are up to 3 % slower).
// One workgroup per compute unit, each with whole units; more where the sums of one would take more than 63 KiB of LDS (64 KiB is
// what a launch gets, and the norm's sums lie beside).
FewPlan few_plan(int M, int N, int K, FewForm form, int cus) {
    const bool quad = M <= 4;
    FewPlan p;
    p.waves = K % 16384 == 0 ? 4 : 8;
    const int longest = (K / PIECE + p.waves - 1) / p.waves;
    const int held = p.waves == 8 && quad ? 8 : 7, most = p.waves == 4 ? 7 : quad ? 8 : 4;
    p.segments = longest <= held ? 1 : (longest + most - 1) / most;
    p.pieces = (longest + p.segments - 1) / p.segments;
    const int units = form == FewForm::plain ? (N + 3) / 4 : N / 8;
    const int per_unit = (form == FewForm::plain ? 1 : 2) * (quad ? 1 : 2) * 16 * p.waves * (int)sizeof(float);
    const int fit = 63 * 1024 / per_unit, rounds = ((units + cus - 1) / cus + fit - 1) / fit;
    p.grid = std::min(units, cus * rounds);
    p.lds = (units + p.grid - 1) / p.grid * per_unit;
    return p;
}

template <int MQ, int P, FewForm FORM, int WAVES>
int launch(const FewTokens& a, const FewPlan& p, hipStream_t st, const CopyJob& beside) {
    const int units = FORM == FewForm::plain ? (a.N + 3) / 4 : a.N / 8;
    auto kern = few_tokens<MQ, P, FORM, WAVES, FewExtra::none>;
    if constexpr (WAVES == 8) {
        if (a.norm) kern = few_tokens<MQ, P, FORM, WAVES, FewExtra::norm>;
        if constexpr (FORM != FewForm::gated) {
            if (beside.blocks) kern = few_tokens<MQ, P, FORM, WAVES, FewExtra::copies>;
            if (a.w_again && !a.norm)
                kern = beside.blocks ? few_tokens<MQ, P, FORM, WAVES, FewExtra::copies, true> : few_tokens<MQ, P, FORM, WAVES, FewExtra::none, true>;
        }
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(p.grid + beside.blocks)), dim3(WAVES * 64), p.lds, st, a, units, p.segments, p.grid, beside);
    KVPR_HIP(hipGetLastError());
    return KVPR_OK;
}

template <int MQ, FewForm FORM, int P>
int launch_pieces(const FewTokens& a, const FewPlan& p, hipStream_t st, const CopyJob& beside) {
    if constexpr (P > 1)
        if (p.pieces < P) return launch_pieces<MQ, FORM, P - 1>(a, p, st, beside);
    return launch<MQ, P, FORM, 8>(a, p, st, beside);
}

template <int MQ, FewForm FORM>
int launch_form(const FewTokens& a, hipStream_t st, const CopyJob& beside) {
    const FewPlan p = few_plan(a.M, a.N, a.K, FORM, compute_units());
    if (p.waves == 4) return launch<MQ, 7, FORM, 4>(a, p, st, beside);     // 32 n pieces a wave, in ceil(32 n / 7) segments: always 7
    return launch_pieces<MQ, FORM, MQ == 1 ? 8 : 7>(a, p, st, beside);
}

}  // namespace

// Up to 8 rows, except where the other kernels are the better ones: 5 rows and more of less than 1024 columns, where the
// launch is all there is (2304 x 768, M = 8: 3.8 us there, 4.0 here), and 7 or 8 rows in several segments of few steps, whose
// ends are not hidden (4096 x 11008, M = 8: 18.5 there, in slices of K, and 19.2 here; 4096 x 16384: 27.5 and 27.4; with 5 rows
// 18.6 and 17.7; 5120 x 13824, five steps: 27.2 and 26.2).
bool few_tokens_along(int M, int N, int K) {
    if (M <= 4) return true;
    if (M > 8 || K < 1024) return false;
    return M <= 6 || K <= 7168 || N > 16 * compute_units();
}

// A product with nothing along: of less than 1024 columns, some waves have one piece of K or none, and the exchange of their sums is
// longer than the read.  There / here, us, M = 1: 768 x 768 3.1 / 3.6, 2304 x 768 3.3 / 3.9, 6144 x 768 4.5 / 4.7, 9216 x 768 6.1 /
// 5.8, 32768 x 768 12.1 / 11.1; 2304 x 256 2.7 / 3.4, 32768 x 256 6.4 / 7.4; 9216 x 640 5.7 / 5.4, 9216 x 512 5.0 / 5.1; of 1024
// columns 2304 x 1024 5.6 / 4.1.  (A launch of its own for what goes along is 4 us.)
bool takes_few_tokens(int M, int N, int K) {
    return few_tokens_along(M, N, K) && (K >= 1024 || (K >= 640 && N > 32 * compute_units()));
}

// x has to be in registers whole: one segment (see few_plan)
bool few_tokens_norm(int M, int N, int K) { return few_tokens_along(M, N, K) && K <= (M <= 4 ? 8192 : 7168); }

int launch_few_tokens(const FewTokens& a, FewForm form, hipStream_t st, const CopyJob& job) {
    // the copies are a launch of their own where no instantiation takes them: with a norm, in the gated form, with 4 waves
    CopyJob beside = job;
    if (a.norm || form == FewForm::gated || a.K % 16384 == 0) {
        if (int rc = launch_copy(job, kCopyThreads, st)) return rc;
        beside = CopyJob();
    }
    auto go = [&](auto f) {
        constexpr FewForm F = decltype(f)::value;
        return a.M <= 4 ? launch_form<1, F>(a, st, beside) : launch_form<2, F>(a, st, beside);
    };
    switch (form) {
        case FewForm::gated: return go(std::integral_constant<FewForm, FewForm::gated>{});
        case FewForm::rotary: return go(std::integral_constant<FewForm, FewForm::rotary>{});
        default: return go(std::integral_constant<FewForm, FewForm::plain>{});
    }
}

}  // namespace kvpr

// for tests: whether the kernel takes a product with something along / alone
extern "C" int kvpr_debug_few_tokens(int M, int N, int K, int alone) { return alone ? kvpr::takes_few_tokens(M, N, K) : kvpr::few_tokens_along(M, N, K); }

// for tests: the cut of a product on a device of `cus` compute units; form 0 plain, 1 gated, 2 rotary
extern "C" int kvpr_debug_few_plan(int M, int N, int K, int form, int cus, int32_t* waves, int32_t* pieces, int32_t* segments, int32_t* grid,
                                   int32_t* lds) {
    const kvpr::FewPlan p = kvpr::few_plan(M, N, K, (kvpr::FewForm)form, cus);
    *waves = p.waves;
    *pieces = p.pieces;
    *segments = p.segments;
    *grid = p.grid;
    *lds = p.lds;
    return KVPR_OK;
}

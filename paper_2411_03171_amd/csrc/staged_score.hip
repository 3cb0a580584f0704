// Staged sweep, first kernel: the scores z of a slab of label rows for a tile
// of samples, the loss, and the dlogits g (Sec. 2.2 gathered forward, the
// appendix's BCE or the squared hinge), with the batch's X images.
//
// A workgroup keeps the X tile in LDS for its whole life and walks a
// contiguous range of rows, 4 per wave and step, with no barrier: 16 lanes
// serve a row, a lane NP (bf16) or SPL (fp32) samples.  The next round of
// indices and weights is in flight while the current one is gathered.
//
// The targets are a bit per sample and row in LDS, for as many rows at a time
// as the image leaves room for: the workgroup takes its rows in segments and
// scans the batch's positives before each.  A label that repeats sets its bit
// twice.  Positives are rare (a few per sample), so a wave whose four rows have
// none takes the loss of a negative without looking at the bits.  (Taking every
// pair as a negative and correcting the positives afterwards cannot give the
// loss and the row sums of g their small values back: the terms of a positive
// with a large score do not cancel to the last bit.)
#include <algorithm>
#include <type_traits>

#include "gather_dev.h"

namespace ffsl {

namespace {

using namespace gdev;

constexpr int SC_MAX_THREADS = 1024;

struct LossGrad {
    float loss, g;
};

// loss and dlogit of a score (y = 0 or 1).  The hardware base-2 exp and log
// and reciprocal with one correction each: exp's argument carries the low part
// of |z| log2(e), the reciprocal takes a Newton step, and the log adds what
// 1 + e lost to rounding, so that a confident negative (e far below 1) still
// contributes its e.
__device__ __forceinline__ LossGrad loss_grad(float z, bool y, int hinge, float s) {
    LossGrad r;
    if (hinge) {
        // squared hinge with yh = 2y - 1
        const float yh = y ? 1.f : -1.f;
        const float hh = fmaxf(1.f - yh * z, 0.f);
        r.loss = hh * hh;
        r.g = -2.f * s * yh * hh;
    } else {
        constexpr float L2E = 1.44269502162933349609375f, L2E_LO = 1.925963033500011079e-8f, LN2 = 0.693147182464599609375f;
        const float az = fabsf(z), t = az * L2E;
        const float lo = fmaf(az, L2E_LO, fmaf(az, L2E, -t));
        const float p = __builtin_amdgcn_exp2f(-t);
        const float e = t < 126.f ? fmaf(p, -LN2 * lo, p) : t != t ? t : 0.f;   // exp(-|z|), 0 below 2^-126
        const float u = 1.f + e;
        float q = __builtin_amdgcn_rcpf(u);
        q = fmaf(fmaf(-u, q, 1.f), q, q);
        // z * 0: an infinite score shows in the loss
        r.loss = (y ? fmaxf(z, 0.f) - z : fmaf(z, 0.f, fmaxf(z, 0.f))) +
                 fmaf(__builtin_amdgcn_logf(u), LN2, (e - (u - 1.f)) * q);
        r.g = s * ((z >= 0.f ? q : e * q) - (y ? 1.f : 0.f));
    }
    return r;
}

// g as bf16 planes: each takes the leading 8 significant bits of what is left
// (exact: three planes hold the 24 bits of an fp32); one plane is rounded.  A
// non-finite g (ODD: there may be one) is all in the first plane.
template <int S, bool ODD>
__device__ __forceinline__ void planes(float g, uint16_t (&p)[S > 0 ? S : 1]) {
    if constexpr (S == 1) {
        p[0] = (uint16_t)(pack_bf16(g, 0.f) & 0xffffu);
    } else if constexpr (S == 3) {
        if (ODD && (__float_as_uint(g) & 0x7f800000u) == 0x7f800000u) {
            p[0] = f32_to_bf16_bits(g);
            p[1] = p[2] = 0;
            return;
        }
        const uint32_t h = __float_as_uint(g) & 0xffff0000u;
        const float r1 = g - __uint_as_float(h);
        const uint32_t m = __float_as_uint(r1) & 0xffff0000u;
        const float r2 = r1 - __uint_as_float(m);
        p[0] = (uint16_t)(h >> 16);
        p[1] = (uint16_t)(m >> 16);
        p[2] = (uint16_t)(__float_as_uint(r2) >> 16);
    }
}

// store the NP consecutive samples NP q .. of row l of every plane
template <int NP, int S, bool ODD>
__device__ __forceinline__ void store_g(Rsrc rG, uint32_t row_elems, int q, bool ok, uint32_t nb_G, const float (&g)[NP]) {
    constexpr uint32_t BT = 16u * NP;
    uint16_t p[NP][S];
#pragma unroll
    for (int e = 0; e < NP; ++e) planes<S, ODD>(g[e], p[e]);
#pragma unroll
    for (int pl = 0; pl < S; ++pl) {
        const uint32_t o = ok ? (row_elems + pl * BT + (uint32_t)(NP * q)) * 2u : nb_G;
        if constexpr (NP == 4) {
            typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
            const u32x2 v = {(uint32_t)p[0][pl] | ((uint32_t)p[1][pl] << 16), (uint32_t)p[2][pl] | ((uint32_t)p[3][pl] << 16)};
            __builtin_amdgcn_raw_buffer_store_b64(v, rG, o, 0, 0);
        } else if constexpr (NP == 2) {
            st32(rG, o, (uint32_t)p[0][pl] | ((uint32_t)p[1][pl] << 16));
        } else {
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)p[0][pl], rG, o, 0, 0);
        }
    }
}

// NP samples per lane; S planes of g (0: none); FULL: bf16 fan-ins that are a
// multiple of 32 (unused for fp32)
template <int VT, int NP, int S, bool FULL, bool IDX16>
__global__ void __launch_bounds__(SC_MAX_THREADS) k_score(const ScoreArgs a) {
    extern __shared__ __align__(16) unsigned char st_smem[];
    constexpr bool BF = VT == FFSL_BF16;
    constexpr int BT = 16 * NP;
    constexpr uint32_t COL = (BF ? 32u : 64u) * NP;
    constexpr uint32_t vsz = BF ? 2u : 4u;
    const int tid = threadIdx.x, lane = tid & 63, nthr = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nwaves = nthr >> 6;
    const int grp = lane >> 4, q = lane & 15;
    const int d = a.d, k = a.k;
    const int tile = blockIdx.y, b0 = tile * BT, nb = min(BT, a.B - b0);
    const uint32_t image = (uint32_t)(d + 1) * COL;
    // after the image: the targets of a segment of rows, a bit per sample
    constexpr int YW = BT == 64 ? 2 : 1;             // words per row
    uint32_t *ym = reinterpret_cast<uint32_t *>(st_smem + image);   // seg_rows * YW
    float *red = reinterpret_cast<float *>(ym);      // one loss sum per wave, at the end

    const uint32_t r0 = blockIdx.x * a.rows_per_wg, r1 = min(a.rows, r0 + a.rows_per_wg);
    const Rsrc rI = make_rsrc(a.I, a.rows * (uint32_t)k * (a.idx16 ? 2u : 4u));
    const Rsrc rW = make_rsrc(a.W, a.rows * (uint32_t)k * vsz);
    const Rsrc rB = make_rsrc(a.bias, a.bias ? a.rows * 4u : 0u);
    const Rsrc rG = make_rsrc(a.G, a.nb_G);
    const uint32_t s_tile = (uint32_t)tile * a.rows;   // gsum elements
    const Rsrc rS = make_rsrc(a.gsum, S > 0 ? (s_tile + a.rows) * 4u : 0u);
    const uint32_t g_tile = (uint32_t)tile * a.rows * (uint32_t)(S * BT);   // elements

    // bf16: a lane reads piece p = e ^ (grp mod NP) of its sample block, so
    // the wave's rows touch different pieces; accumulator e is sample NP q + p
    const int gx = grp & (NP - 1);
    const uint32_t pbase = BF ? 8u * NP * (q & 3) + 8u * gx : 0u;

    const int rounds = (k + 31) >> 5;
    const uint32_t step = 4u * nwaves;
    uint32_t l_cur = r0 + 4u * wave, l_nxt = l_cur;
    int rd_cur = 0, rd_nxt = 0;
    auto advance = [&](uint32_t &l, int &rd) {
        if (++rd == rounds) {
            rd = 0;
            l += step;
        }
    };
    using Rd = typename std::conditional<BF, TrRound<FULL>, FRound>::type;
    auto load = [&](Rd &o, float &bias) {
        const uint32_t l = l_nxt + grp;   // rows past the slab read zeros
        if constexpr (BF)
            tr_load_round<FULL, IDX16>(rI, rW, l, k, rd_nxt, q, o);
        else
            f_load_round(rI, rW, l, k, rd_nxt, q, a.idx16, o);
        bias = ldf(rB, l * 4u);
        advance(l_nxt, rd_nxt);
    };

    auto clear_targets = [&] {
        for (uint32_t i = tid; i < a.seg_rows * YW; i += nthr) ym[i] = 0u;
    };
    uint32_t s0 = r0;   // first row of the segment
    auto set_targets = [&](int2 first) {
        const uint32_t n = min(a.seg_rows, r1 - s0);
        for (int base = 0; base < a.nnz; base += nthr) {
            int2 p = first;
            if (base > 0) p = base + tid < a.nnz ? a.pos[base + tid] : make_int2(-1, 0);
            const int64_t lr = (int64_t)p.x - a.row0 - s0;
            const int b = p.y - b0;
            if (lr >= 0 && lr < (int64_t)n && b >= 0 && b < nb) atomicOr(&ym[lr * YW + (b >> 5)], 1u << (b & 31));
        }
    };

    // the first positives and the next two rounds load while the tile is staged
    const int2 mypos = tid < a.nnz ? a.pos[tid] : make_int2(-1, 0);
    Rd ra, rb;
    float ba, bb;
    load(ra, ba);
    load(rb, bb);
    clear_targets();
    stage_image(a.xa + (size_t)tile * image, image, wave, lane, nwaves);
    __syncthreads();

    float loss_acc = 0.f;
    float z[NP];
#pragma unroll
    for (int e = 0; e < NP; ++e) z[e] = 0.f;

    auto process = [&](const Rd &o, float bias) {
        const int kr = k - 32 * rd_cur;
        // the targets of the lane's samples
        uint32_t yw = 0u;
        if (rd_cur == rounds - 1) yw = ym[(l_cur + grp - s0) * YW + (BT == 64 ? q >> 3 : 0)];
        if constexpr (BF)
            tr_round<NP, FULL>(o, d, kr, q, pbase, z);
        else
            f_round<NP>(o, d, kr, q, (uint32_t)q * NP * 4u, z);
        if (rd_cur == rounds - 1) {
            const uint32_t l = l_cur + grp;
            const bool valid = l < r1;
            float zs[NP];   // in sample order
#pragma unroll
            for (int e = 0; e < NP; ++e) zs[e] = z[e] + bias;
            if constexpr (BF && NP >= 2) {
#pragma unroll
                for (int e = 0; e < NP; e += 2) {
                    const float x = zs[e], y = zs[e + 1];
                    zs[e] = (gx & 1) ? y : x;
                    zs[e + 1] = (gx & 1) ? x : y;
                }
            }
            if constexpr (BF && NP == 4) {
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const float x = zs[e], y = zs[e + 2];
                    zs[e] = (gx & 2) ? y : x;
                    zs[e + 2] = (gx & 2) ? x : y;
                }
            }
            if (a.logits) {
#pragma unroll
                for (int e = 0; e < NP; ++e)
                    if (valid && NP * q + e < nb)
                        a.logits[(int64_t)(b0 + NP * q + e) * a.L + a.row0 + l] = zs[e];
            }
            // every pair as a negative; where one is a positive or has a g that is
            // not finite, the wave's pairs once more
            const uint32_t y = (yw >> (NP * q & 31)) & ((1u << NP) - 1u);
            float g[NP], sg, ls;
            auto grads = [&](auto odd) {
                sg = ls = 0.f;
#pragma unroll
                for (int e = 0; e < NP; ++e) {
                    const bool live = valid && NP * q + e < nb;
                    const LossGrad r = loss_grad(zs[e], odd && ((y >> e) & 1u), a.hinge, a.s);
                    ls += live ? r.loss : 0.f;
                    g[e] = live ? r.g : 0.f;
                    sg += g[e];
                }
            };
            auto store = [&](auto odd) {
                if constexpr (S > 0)
                    store_g<NP, S, decltype(odd)::value>(rG, g_tile + l * (uint32_t)(S * BT), q, valid, a.nb_G, g);
            };
            grads(std::false_type{});
            if (__builtin_amdgcn_ballot_w64(y != 0u || (S == 3 && (__float_as_uint(sg) & 0x7f800000u) == 0x7f800000u)) == 0) {
                store(std::false_type{});
            } else {
                grads(std::true_type{});
                store(std::true_type{});
            }
            loss_acc += ls;
            if constexpr (S > 0) {
                sg = sum16(sg);
                stf(rS, valid && q == 0 ? (s_tile + l) * 4u : 0xfffffff0u, sg);
            }
#pragma unroll
            for (int e = 0; e < NP; ++e) z[e] = 0.f;
        }
        advance(l_cur, rd_cur);
    };

    // a whole segment is an even number of steps for every wave, so that it
    // ends on the same of the two rounds in flight
    for (;;) {
        set_targets(mypos);
        __syncthreads();
        const uint32_t s1 = min(r1, s0 + a.seg_rows);
        while (l_cur < s1) {
            process(ra, ba);
            load(ra, ba);
            if (l_cur >= s1) break;
            process(rb, bb);
            load(rb, bb);
        }
        s0 += a.seg_rows;
        if (s0 >= r1) break;
        __syncthreads();
        clear_targets();
        __syncthreads();
    }

    if (a.want_loss) {
        // lanes, then waves, in a fixed order
#pragma unroll
        for (int sh = 32; sh >= 1; sh >>= 1) loss_acc += __shfl_xor(loss_acc, sh);
        __syncthreads();
        if (lane == 0) red[wave] = loss_acc;
        __syncthreads();
        if (tid == 0) {
            float t = red[0];
            for (int w = 1; w < nwaves; ++w) t += red[w];
            const int i = (int)(blockIdx.y * gridDim.x + blockIdx.x);
            a.loss_part[i] = i < a.loss_have ? a.loss_part[i] + t : t;
        }
    }
}

// The X images of the batch (see staged.h) and its positives: one 16-byte word per thread and
// iteration; consecutive lanes take consecutive columns, so the reads of X
// are coalesced.
template <int VT, int NP>
__device__ __forceinline__ uint4 image_a_word(const StagedPrepArgs &a, int tile, int c, int w) {
    constexpr int BT = 16 * NP;
    uint4 r = make_uint4(0u, 0u, 0u, 0u);
    if (c >= a.d) return r;
    uint32_t *o = reinterpret_cast<uint32_t *>(&r);
    const int b0 = tile * BT;
    if constexpr (VT == FFSL_BF16) {
        const uint16_t *X = static_cast<const uint16_t *>(a.X);
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int sp = 2 * w + (i >> 2);   // stored 8-byte piece
            const int m = sp / NP, p = (sp % NP) ^ staged_swz_a(c, NP);
            const int b = b0 + NP * (4 * m + (i & 3)) + p;
            const uint32_t x = b < a.B ? X[(size_t)b * a.d + c] : 0u;
            o[i >> 1] |= x << (16 * (i & 1));
        }
    } else {
        const float *X = static_cast<const float *>(a.X);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int b = b0 + 4 * w + i;
            o[i] = b < a.B ? __float_as_uint(X[(size_t)b * a.d + c]) : 0u;
        }
    }
    return r;
}

template <int VT, int BTW>
__device__ __forceinline__ uint4 image_b_word(const StagedPrepArgs &a, int tile, int c, int w) {
    using Im = DwImage<VT, BTW>;
    uint4 r = make_uint4(0u, 0u, 0u, 0u);
    uint32_t *o = reinterpret_cast<uint32_t *>(&r);
    const int P = Im::place(w, c), oct = Im::octet(P), pl = Im::plane(P);   // the swizzle is its own inverse
    if (oct < 0) return r;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int b = tile * BTW + 8 * oct + i;
        uint32_t x = 0u;
        if (b < a.B) {
            if constexpr (VT == FFSL_BF16) {
                x = static_cast<const uint16_t *>(a.X)[(size_t)b * a.d + c];
            } else {
                // plane pl of the value's three bf16 planes (exact; a non-finite
                // value is all in the first)
                float f = static_cast<const float *>(a.X)[(size_t)b * a.d + c];
                if ((__float_as_uint(f) & 0x7f800000u) == 0x7f800000u) {
                    x = pl == 0 ? f32_to_bf16_bits(f) : 0u;
                } else {
                    for (int t = 0; t < pl; ++t) f -= __uint_as_float(__float_as_uint(f) & 0xffff0000u);
                    x = __float_as_uint(f) >> 16;
                }
            }
        }
        o[i >> 1] |= x << (16 * (i & 1));
    }
    return r;
}

template <int VT, int NP, int BTW>
__global__ void __launch_bounds__(256) k_staged_prep(const StagedPrepArgs a) {
    constexpr int WA = (VT == FFSL_BF16 ? 32 : 64) * NP / 16, WB = DwImage<VT, BTW>::COL / 16;
    const int64_t na = (int64_t)a.p.tiles * WA * (a.d + 1);
    const int64_t nimg = na + (a.xb ? (int64_t)a.p.tilesw * WB * a.d : 0);
    const int64_t npos = nimg + a.nnz, nall = npos + a.nzero;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < nall; i += (int64_t)gridDim.x * 256) {
        if (i < na) {
            const int c = (int)(i % (a.d + 1)), tw = (int)(i / (a.d + 1));
            reinterpret_cast<uint4 *>(a.xa)[((int64_t)(tw / WA) * (a.d + 1) + c) * WA + tw % WA] =
                image_a_word<VT, NP>(a, tw / WA, c, tw % WA);
        } else if (i < nimg) {
            const int64_t n = i - na;
            const int c = (int)(n % a.d), tw = (int)(n / a.d);
            reinterpret_cast<uint4 *>(a.xb)[((int64_t)(tw / WB) * a.d + c) * WB + tw % WB] =
                image_b_word<VT, BTW>(a, tw / WB, c, tw % WB);
        } else if (i >= npos) {
            a.zero[i - npos] = 0u;
        } else {
            // a positive's sample is the last b with off[b] <= e
            const int e = (int)(i - nimg), lb = a.lab[e];
            int lo = 0, hi = a.B - 1;
            while (lo < hi) {
                const int mid = (lo + hi + 1) >> 1;
                if (a.off[mid] <= e) lo = mid;
                else hi = mid - 1;
            }
            const bool ok = lb >= 0 && a.off[lo] <= e && e < a.off[lo + 1];
            a.pos[e] = make_int2(ok ? lb : -1, lo);
        }
    }
}

typedef void (*ScoreKernel)(const ScoreArgs);
template <int VT, int NP, int S>
ScoreKernel score_s(bool full, bool idx16) {
    if constexpr (VT == FFSL_F32)
        return k_score<VT, NP, S, false, false>;
    else if constexpr (S == 1)   // fan-in 32 and 64 only
        return idx16 ? k_score<VT, NP, S, true, true> : k_score<VT, NP, S, true, false>;
    else
        return full ? (idx16 ? k_score<VT, NP, S, true, true> : k_score<VT, NP, S, true, false>)
                    : (idx16 ? k_score<VT, NP, S, false, true> : k_score<VT, NP, S, false, false>);
}
template <int VT, int NP>
ScoreKernel score_np(int S, bool full, bool idx16) {
    if (S == 0) return score_s<VT, NP, 0>(full, idx16);
    // one plane: batches that a fused fast path does not take, of 17 samples at
    // least
    if constexpr (VT == FFSL_BF16 && NP >= 2)
        if (S == 1) return score_s<VT, NP, 1>(full, idx16);
    return score_s<VT, NP, 3>(full, idx16);
}

size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

size_t staged_xa_bytes(int32_t d, int32_t vt, int32_t B_max) {
    return al256((size_t)(B_max + 63) * (size_t)(d + 1) * (vt == FFSL_BF16 ? 2 : 4));
}
size_t staged_xb_bytes(int32_t d, int32_t vt, int32_t B_max) {
    return al256((size_t)(B_max + 63) * (size_t)d * (vt == FFSL_BF16 ? 2 : 8));
}
// G holds at least one step of rows for the largest batch, and STAGED_G_MAX
// bytes in full
size_t staged_g_bytes(int64_t L, int32_t B_max) {
    const int64_t per_row = (int64_t)(B_max + 63) * 3 * 2, rows = (L + 63) / 64 * 64;
    return al256((size_t)std::min<int64_t>(rows, std::max<int64_t>((STAGED_G_MAX + per_row - 1) / per_row, 64)) * (size_t)per_row);
}

// a sum per (tile, row) of G, whose tiles hold 16 samples and min_S planes at
// least
size_t staged_gsum_bytes(int64_t L, int32_t B_max, int min_S) {
    return al256((size_t)std::min<int64_t>((L + 63) / 64 * 64 * ((B_max + 15) / 16), (int64_t)(staged_g_bytes(L, B_max) / (32 * min_S))) * 4);
}

StagedPlan staged_plan(const Layer &ly, int B, int S, size_t g_bytes) {
    StagedPlan p{};
    const bool bf = ly.vt == FFSL_BF16;
    // the widest tile whose image fits 144 KiB of LDS, and no wider than the
    // batch needs
    const int most = bf ? 64 : 32;
    int BT = B <= 16 ? 16 : B <= 32 ? 32 : most;
    BT = std::min(BT, most);
    while (BT > 16 && (size_t)(ly.d + 1) * BT * (bf ? 2 : 4) > 144 * 1024) BT /= 2;
    p.BT = BT;
    p.BTW = BT;
    if (!bf && p.BTW == 32 && (size_t)ly.d * 192 > 152 * 1024) p.BTW = 16;
    if (!bf && p.BTW == 16 && (size_t)ly.d * 128 > 152 * 1024) p.BTW = 8;
    p.tiles = (B + BT - 1) / BT;
    p.tilesw = (B + p.BTW - 1) / p.BTW;
    p.S = S;
    p.cola = BT * (bf ? 2 : 4);
    p.colb = bf ? 2 * p.BTW : p.BTW == 32 ? 192 : p.BTW == 16 ? 128 : 64;
    int64_t most_rows = STAGED_SLAB_ROWS;
    if (S > 0) most_rows = std::min<int64_t>(most_rows, (int64_t)(g_bytes / ((size_t)p.tiles * BT * S * 2)) / 64 * 64);
    // slabs of equal size: a small remainder costs three launches that each stage
    // their image again (about 52 us of a step of 1048576 rows, fan-in 64, d 2048,
    // B 128, whose third slab had 128 rows)
    const int64_t slabs = (ly.L + most_rows - 1) / most_rows;
    const int64_t even = (ly.L + slabs - 1) / slabs;
    // whole steps of 16 waves on every CU where that leaves as many slabs: the
    // last step of seven slabs of 149797 rows was a ninth full
    const int64_t unit = (int64_t)ly.num_cu * 64, whole = (even + unit - 1) / unit * unit;
    p.slab = slabs > 1 && whole <= most_rows ? whole : (even + 63) / 64 * 64;
    return p;
}

int launch_staged_prep(const Layer &ly, const StagedPrepArgs &a, hipStream_t st) {
    const int64_t n = (int64_t)a.p.tiles * (a.p.cola / 16) * (a.d + 1) +
                      (a.xb ? (int64_t)a.p.tilesw * (a.p.colb / 16) * a.d : 0) + a.nnz + a.nzero;
    const dim3 grid((unsigned)std::min<int64_t>((n + 255) / 256, 2048)), blk(256);
#define FFSL_PREP(VT, NP, BTW) hipLaunchKernelGGL((k_staged_prep<VT, NP, BTW>), grid, blk, 0, st, a)
    if (ly.vt == FFSL_BF16) {
        if (a.p.BT == 64) FFSL_PREP(FFSL_BF16, 4, 64);
        else if (a.p.BT == 32) FFSL_PREP(FFSL_BF16, 2, 32);
        else FFSL_PREP(FFSL_BF16, 1, 16);
    } else if (a.p.BT == 32) {
        if (a.p.BTW == 32) FFSL_PREP(FFSL_F32, 2, 32);
        else if (a.p.BTW == 16) FFSL_PREP(FFSL_F32, 2, 16);
        else FFSL_PREP(FFSL_F32, 2, 8);
    } else {
        if (a.p.BTW == 16) FFSL_PREP(FFSL_F32, 1, 16);
        else FFSL_PREP(FFSL_F32, 1, 8);
    }
#undef FFSL_PREP
    return check_launch("staged_prep");
}

int launch_score(const Layer &ly, const StagedPlan &p, ScoreArgs &a, int *nwg_out, hipStream_t st) {
    const bool full = ly.k % 32 == 0, i16 = ly.idx16 != 0;
    const int NP = p.BT / 16;
    ScoreKernel kern;
    if (ly.vt == FFSL_BF16)
        kern = NP == 4 ? score_np<FFSL_BF16, 4>(p.S, full, i16)
             : NP == 2 ? score_np<FFSL_BF16, 2>(p.S, full, i16) : score_np<FFSL_BF16, 1>(p.S, full, i16);
    else
        kern = NP == 2 ? score_np<FFSL_F32, 2>(p.S, full, i16) : score_np<FFSL_F32, 1>(p.S, full, i16);
    // workgroups of 4 to 16 waves: as many waves as give every CU work, and 16
    // only where the rows feed them
    int waves = 16;
    while (waves > 4 && (int64_t)a.rows < (int64_t)ly.num_cu * 4 * waves) waves /= 2;
    const size_t image = (size_t)(ly.d + 1) * p.cola, lds = 160 * 1024;
    const int occ = std::max(1, std::min(2, (int)(lds / (image + 12 * 1024))));
    int64_t nwg = std::min<int64_t>((int64_t)ly.num_cu * occ, (a.rows + 4 * waves - 1) / (4 * waves));
    nwg = std::min<int64_t>(nwg, ly.max_parts);
    const int64_t per = (a.rows + nwg - 1) / nwg;
    a.rows_per_wg = (uint32_t)((per + 4 * waves - 1) / (4 * waves) * (4 * waves));
    nwg = (a.rows + a.rows_per_wg - 1) / a.rows_per_wg;
    // the targets of as many rows as fit: a multiple of two steps of every wave
    const size_t per_row = p.BT == 64 ? 8 : 4, unit = 8 * waves;
    const size_t want = (a.rows_per_wg + unit - 1) / unit * unit, room = (lds / occ - image) / per_row / unit * unit;
    a.seg_rows = (uint32_t)std::min(want, room);
    const size_t shm = image + a.seg_rows * per_row;
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(kern),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)shm);
    if (e != hipSuccess) return fail(FFSL_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
    hipLaunchKernelGGL(kern, dim3((unsigned)nwg, p.tiles), dim3(waves * 64), shm, st, a);
    *nwg_out = (int)nwg;
    return check_launch("score");
}

}  // namespace ffsl

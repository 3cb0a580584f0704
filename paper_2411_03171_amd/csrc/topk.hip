// Inference over the label space: the scores of a batch against every label
// row (the gathered forward of Sec. 2.2) and, per sample, the labels with the
// highest scores -- the prediction that Precision@k scores (appendix on
// evaluation metrics).  The scores never reach memory.
//
// k_topk_any    The scan for bf16 values (below).
// k_topk_scan   The scan for fp32 values.  One persistent workgroup per CU
//               slot and batch tile.  The X tile is staged in LDS as
//               [d+1][BT] (column d is zero).  A wave serves 4 label rows at
//               a time, one per DPP row of 16 lanes; a lane serves SPL
//               consecutive samples of the tile.  In each round of 32 slots,
//               lane u loads slots 2u and 2u+1 of its row, and row_newbcast
//               hands every slot pair to all 16 lanes of the row, which
//               gather their samples' X values from LDS.
//               Both scans: each lane keeps, per sample, the KP best (score,
//               label) keys it has seen, sorted, in registers; a new key is
//               inserted only when it beats the last one and the bounds that
//               the other lists set.  At the end the workgroup merges its
//               lists per sample into one and writes it out.
// k_topk_merge  One workgroup per sample merges the lists of all
//               workgroups: K rounds of a block-wide maximum over the heads
//               of the sorted lists.  Writes labels, scores and relevance.
// k_patk        Precision@k averaged over the batch.
//
// Order of the result: descending score, equal scores by ascending label;
// NaN scores are never selected.  A (score, label) pair is one 64-bit key
// that orders exactly that way, so lists compare with one integer compare.

#include <mutex>

#include "gather_dev.h"

// Scratch of the no-allocation inference call (ffsl_infer_topk_noalloc): the
// same workspace layout as ffsl_infer_topk's, in a file-scope device array
// that each GPU the library runs on holds until the process ends.  Host code
// never uses this name as an address: the device address comes from
// hipGetSymbolAddress, once per device (topk_scratch below).  Nothing in it
// needs to start at zero: the scan writes every list the merge reads, and the
// merge every relevance flag the P@k kernel reads.
// The array has external linkage (and default visibility): with internal
// linkage the device code object keeps it as a local symbol, which the
// runtime's symbol lookup cannot find.
__device__ __align__(256) __attribute__((visibility("default"))) unsigned char
    ffsl_topk_scratch[FFSL_TOPK_SCRATCH_BYTES];

namespace ffsl {

namespace {
constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex g_scratch_mu;
void *g_scratch[SCRATCH_MAX_DEVICES];   // device address of `scratch` per device
}  // namespace

int topk_scratch(int device, char **ptr) {
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return fail(FFSL_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
    if (cur != device)
        return fail(FFSL_EINVAL, "the layer lives on device %d but device %d is current", device, cur);
    if (device < 0 || device >= SCRATCH_MAX_DEVICES)
        return fail(FFSL_EUNSUPPORTED, "device %d: the no-allocation call supports devices 0..%d", device,
                    SCRATCH_MAX_DEVICES - 1);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch[device]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(ffsl_topk_scratch));
        if (e != hipSuccess || !p)
            return fail(FFSL_EHIP, "hipGetSymbolAddress(ffsl_topk_scratch): %s", hipGetErrorString(e));
        g_scratch[device] = p;
    }
    *ptr = static_cast<char *>(g_scratch[device]);
    return FFSL_OK;
}
namespace {
using namespace fdev;

constexpr int TK_THREADS = 512;
constexpr int TK_WAVES = TK_THREADS / 64;
constexpr int TK_ROWS = 4;                     // label rows per wave per step
constexpr int TK_LISTS = TK_WAVES * TK_ROWS;   // lists per sample in a workgroup
constexpr int TK_SHARE = 64;                   // workgroups that publish their bests (k_topk_any)
constexpr int TK_MERGE_THREADS = 256;
constexpr int TK_AHEAD = 8;                    // steps of row data loaded ahead
constexpr int DPP_ROW_NEWBCAST = 0x150;        // + n: lane n of each DPP row to the whole row

struct TkArgs {
    const void *X;
    const void *W;
    const int32_t *I;
    const float *bias;
    int64_t L;
    int32_t B, d, k;
    int32_t nwg;       // workgroups per batch tile (gridDim.x)
    int32_t thr_off;   // LDS byte offset of the per-sample shared bounds, then
                       // of the best score of each of the lists per sample
    int32_t K;         // labels wanted per sample
    int32_t idx16;     // I holds uint16 indices
    uint64_t *part;    // [B][nwg][KP] keys, sorted descending per list
    const unsigned char *xa;   // k_topk_any: X images (staged.h), or null
    int64_t rows_per_wg;       // k_topk_any: consecutive rows of a workgroup
    uint32_t *best;            // k_topk_any: [B][TK_SHARE] best score of a workgroup so far, or null
};

// (score, label) as an integer ordered like (score descending, label
// ascending): the score's bits mapped to an order-preserving unsigned value
// (with -0 taken as +0) in the high word, the complemented label in the low
// word.  Key 0 marks an empty entry; no scored label maps to it.
__device__ __forceinline__ uint64_t score_key(float z, uint32_t l) {
    uint32_t u = __float_as_uint(z);
    u = u == 0x80000000u ? 0u : u;
    u ^= (u & 0x80000000u) ? 0xffffffffu : 0x80000000u;
    return ((uint64_t)u << 32) | (uint64_t)(~l);
}

// the score of a key (-inf for the empty key 0)
__device__ __forceinline__ float key_score(uint64_t key) {
    const uint32_t u = (uint32_t)(key >> 32);
    return u == 0u ? -INFINITY : __uint_as_float((u & 0x80000000u) ? (u ^ 0x80000000u) : ~u);
}

__device__ __forceinline__ int32_t key_label(uint64_t key) { return key ? (int32_t)(~(uint32_t)key) : -1; }

// Insert nk into the descending list kl, dropping the last entry; nk must
// beat kl[KP-1].
template <int KP>
__device__ __forceinline__ void list_insert(uint64_t (&kl)[KP], uint64_t nk) {
    bool lt[KP];
#pragma unroll
    for (int p = 0; p < KP; ++p) lt[p] = kl[p] < nk;
#pragma unroll
    for (int p = KP - 1; p > 0; --p) kl[p] = lt[p - 1] ? kl[p - 1] : (lt[p] ? nk : kl[p]);
    kl[0] = lt[0] ? nk : kl[0];
}

// Merge the sorted list src[0..KP) (in memory) into kl: entries are taken in
// order until one does not beat kl's last.
template <int KP, typename P>
__device__ __forceinline__ void list_merge(uint64_t (&kl)[KP], const P *src) {
    for (int p = 0; p < KP; ++p) {
        const uint64_t key = src[p];
        if (key <= kl[KP - 1]) break;
        list_insert(kl, key);
    }
}

// row data of one round for this lane as loaded: the columns of its two
// slots (d for a slot past k: column d of the tile is zero), the two weights
// and, in round 0, the row's bias.  Converted to LDS offsets only where used,
// so the loads of the next step stay in flight.
struct TkRaw {
    int2 c;
    float2 w;
    float bias;
};

__device__ __forceinline__ void tk_load(const TkArgs &a, int64_t l0, int r, int g, int u, TkRaw &out) {
    const int64_t l = min(l0 + g, a.L - 1);
    const int s0 = 32 * r + 2 * u;
    const int64_t base = l * a.k;
    const float *W = static_cast<const float *>(a.W);
    if ((a.k & 1) == 0) {
        // even fan-in: the pair is two word loads (the same word twice with
        // 16-bit indices) and one load of the weights
        if (s0 < a.k) {
            const uint32_t ish = a.idx16 ? 1u : 2u;
            const char *ip = reinterpret_cast<const char *>(a.I) + ((size_t)(base + s0) << ish);
            out.c.x = *reinterpret_cast<const int32_t *>(ip);
            out.c.y = *reinterpret_cast<const int32_t *>(ip + (a.idx16 ? 0 : 4));
            out.w = *reinterpret_cast<const float2 *>(W + base + s0);
        } else {
            out.c = a.idx16 ? make_int2(a.d | (a.d << 16), 0) : make_int2(a.d, a.d);
            out.w = make_float2(0.f, 0.f);
        }
    } else {
        // odd fan-in: the two slots are loaded one by one and packed as an
        // even fan-in's pair would be
        const uint16_t *I16 = reinterpret_cast<const uint16_t *>(a.I);
        if (a.idx16) {
            const uint32_t c0 = s0 < a.k ? I16[base + s0] : (uint32_t)a.d;
            const uint32_t c1 = s0 + 1 < a.k ? I16[base + s0 + 1] : (uint32_t)a.d;
            out.c = make_int2((int)(c0 | (c1 << 16)), 0);
        } else {
            out.c.x = s0 < a.k ? a.I[base + s0] : a.d;
            out.c.y = s0 + 1 < a.k ? a.I[base + s0 + 1] : a.d;
        }
        out.w = make_float2(s0 < a.k ? W[base + s0] : 0.f, s0 + 1 < a.k ? W[base + s0 + 1] : 0.f);
    }
    out.bias = (r == 0 && a.bias) ? a.bias[l] : 0.f;
}

// LDS offsets and weights of a round, ready for the broadcasts
struct TkRound {
    int32_t o0, o1;
    float2 w;
};

template <int SPL>
__device__ __forceinline__ TkRound tk_prep(const TkRaw &raw, int d, int idx16) {
    constexpr int COL = 16 * SPL * (int)sizeof(float);   // bytes per LDS column
    // 16-bit indices: one word holds both slots
    const uint32_t r0 = idx16 ? ((uint32_t)raw.c.x & 0xffffu) : (uint32_t)raw.c.x;
    const uint32_t r1 = idx16 ? ((uint32_t)raw.c.x >> 16) : (uint32_t)raw.c.y;
    // indices outside [0,d) are clamped (the layer's precondition excludes
    // them); d itself is the zero column
    const uint32_t c0 = min(r0, (uint32_t)d), c1 = min(r1, (uint32_t)d);
    TkRound t;
    t.o0 = (int32_t)c0 * COL;
    t.o1 = (int32_t)c1 * COL;
    t.w = raw.w;
    return t;
}

template <int CTRL>
__device__ __forceinline__ int32_t bcast(int32_t x) {
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true);
}

template <int SPL>
struct TkGather;
template <> struct TkGather<4> { using G = float4; };
template <> struct TkGather<2> { using G = float2; };
template <> struct TkGather<1> { using G = float; };

// z[e] += w0 * xa[e] + w1 * xb[e] for the lane's samples
template <int SPL>
__device__ __forceinline__ void tk_fma(typename TkGather<SPL>::G xa, typename TkGather<SPL>::G xb, float2 w,
                                       float (&z)[SPL]) {
    const float *pa = reinterpret_cast<const float *>(&xa);
    const float *pb = reinterpret_cast<const float *>(&xb);
#pragma unroll
    for (int e = 0; e < SPL; ++e) z[e] = fmaf(w.y, pb[e], fmaf(w.x, pa[e], z[e]));
}

template <int N>
__device__ __forceinline__ float2 bcast_w(float2 w) {
    return make_float2(__int_as_float(bcast<DPP_ROW_NEWBCAST + N>(__float_as_int(w.x))),
                       __int_as_float(bcast<DPP_ROW_NEWBCAST + N>(__float_as_int(w.y))));
}

// slot pair N of the round (loaded by lane N of the row): gather this lane's
// samples of the two columns and accumulate
template <int SPL, int N>
__device__ __forceinline__ void tk_pair(const TkRound &c, int xl, float (&z)[SPL]) {
    using G = typename TkGather<SPL>::G;
    extern __shared__ __align__(16) unsigned char tk_smem[];
    const G xa = *reinterpret_cast<const G *>(tk_smem + (xl + bcast<DPP_ROW_NEWBCAST + N>(c.o0)));
    const G xb = *reinterpret_cast<const G *>(tk_smem + (xl + bcast<DPP_ROW_NEWBCAST + N>(c.o1)));
    tk_fma<SPL>(xa, xb, bcast_w<N>(c.w), z);
}

// the round's slot pairs N .. npairs-1 of a partial round (npairs is uniform)
template <int SPL, int N = 0>
__device__ __forceinline__ void tk_round_part(const TkRound &c, int xl, int npairs, float (&z)[SPL]) {
    if constexpr (N < 16) {
        if (N < npairs) {
            tk_pair<SPL, N>(c, xl, z);
            tk_round_part<SPL, N + 1>(c, xl, npairs, z);
        }
    }
}

// all 16 slot pairs: every gather is issued first, so that they are all in
// flight together, then the products
template <int SPL, int N = 0>
__device__ __forceinline__ void tk_gather_all(const TkRound &c, int xl, typename TkGather<SPL>::G (&xa)[16],
                                              typename TkGather<SPL>::G (&xb)[16]) {
    if constexpr (N < 16) {
        using G = typename TkGather<SPL>::G;
        extern __shared__ __align__(16) unsigned char tk_smem[];
        xa[N] = *reinterpret_cast<const G *>(tk_smem + (xl + bcast<DPP_ROW_NEWBCAST + N>(c.o0)));
        xb[N] = *reinterpret_cast<const G *>(tk_smem + (xl + bcast<DPP_ROW_NEWBCAST + N>(c.o1)));
        tk_gather_all<SPL, N + 1>(c, xl, xa, xb);
    }
}

template <int SPL, int N = 0>
__device__ __forceinline__ void tk_fma_all(const TkRound &c, const typename TkGather<SPL>::G (&xa)[16],
                                           const typename TkGather<SPL>::G (&xb)[16], float (&z)[SPL]) {
    if constexpr (N < 16) {
        tk_fma<SPL>(xa[N], xb[N], bcast_w<N>(c.w), z);
        tk_fma_all<SPL, N + 1>(c, xa, xb, z);
    }
}

template <int SPL>
__device__ __forceinline__ void tk_round_full(const TkRound &c, int xl, float (&z)[SPL]) {
    typename TkGather<SPL>::G xa[16], xb[16];
    tk_gather_all<SPL>(c, xl, xa, xb);
    tk_fma_all<SPL>(c, xa, xb, z);
}

// Stage the batch tile transposed, Xs[c*BT + b], with a zero column d and
// zero samples past B, and clear the per-sample bounds and list bests.
template <int BT>
__device__ __forceinline__ void tk_stage(const TkArgs &a, int b0, int nb) {
    extern __shared__ __align__(16) unsigned char tk_smem[];
    const int tid = threadIdx.x, d = a.d;
    float *Xs = reinterpret_cast<float *>(tk_smem);
    const float *X = static_cast<const float *>(a.X) + (int64_t)b0 * d;
    for (int b = 0; b < BT; ++b)
        for (int c = tid; c <= d; c += TK_THREADS) Xs[c * BT + b] = (b < nb && c < d) ? X[(int64_t)b * d + c] : 0.f;
    for (int i = tid; i < BT * (1 + TK_LISTS); i += TK_THREADS)
        reinterpret_cast<uint32_t *>(tk_smem + a.thr_off)[i] = 0u;
    __syncthreads();
}

// Every wave turns the list bests of BT/8 samples into bounds: the K-th
// largest of a sample's list bests (K distinct labels reach it).
template <int KP, int BT>
__device__ __forceinline__ void tk_list_bound(const uint32_t *lmax, uint32_t *shared_thr, int K, int wave,
                                              int lane) {
    constexpr int PER = BT / TK_WAVES;
    if (lane < PER) {
        const int bt = wave * PER + lane;
        uint32_t best[KP];
#pragma unroll
        for (int p = 0; p < KP; ++p) best[p] = 0u;
        for (int i = 0; i < TK_LISTS; ++i) {
            uint32_t v = __hip_atomic_load(lmax + bt * TK_LISTS + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#pragma unroll
            for (int p = 0; p < KP; ++p) {
                const uint32_t hi = max(best[p], v), lo = min(best[p], v);
                best[p] = hi;
                v = lo;
            }
        }
        uint32_t vk = 0u;
#pragma unroll
        for (int p = 0; p < KP; ++p) vk = p == K - 1 ? best[p] : vk;
        atomicMax(shared_thr + bt, vk);
    }
}

// The workgroup's lists per sample, written to LDS as Ls[bt][list][KP],
// merged into one per sample and written to a.part: four threads per sample
// take a quarter each, one joins the four.  (With one thread joining all, a
// small call, 30000 labels of fan-in 32, B 16, top 8, took 85 us; now 37.)
template <int KP, int BT, int TH = TK_THREADS>
__device__ __forceinline__ void tk_merge_lists(const TkArgs &a, int b0, int nb) {
    extern __shared__ __align__(16) unsigned char tk_smem[];
    uint64_t *Ls = reinterpret_cast<uint64_t *>(tk_smem);
    constexpr int LISTS = TH / 16;
    static_assert(4 * BT <= TH, "four threads per sample");
    __syncthreads();
    const int bt = threadIdx.x >> 2, sub = threadIdx.x & 3;
    uint64_t m[KP];
#pragma unroll
    for (int p = 0; p < KP; ++p) m[p] = 0;
    if (bt < nb) {
        for (int i = 0; i < LISTS / 4; ++i) list_merge(m, Ls + ((size_t)bt * LISTS + sub * (LISTS / 4) + i) * KP);
    }
    __syncthreads();
    if (bt < nb) {
#pragma unroll
        for (int p = 0; p < KP; ++p) Ls[((size_t)bt * LISTS + sub) * KP + p] = m[p];
    }
    __syncthreads();
    if (sub == 0 && bt < nb) {
        for (int i = 1; i < 4; ++i) list_merge(m, Ls + ((size_t)bt * LISTS + i) * KP);
        uint64_t *dst = a.part + ((size_t)(b0 + bt) * a.nwg + blockIdx.x) * KP;
#pragma unroll
        for (int p = 0; p < KP; ++p) dst[p] = m[p];
    }
}

template <int SPL, int KP>
__global__ __launch_bounds__(TK_THREADS) void k_topk_scan(TkArgs a) {
    extern __shared__ __align__(16) unsigned char tk_smem[];
    constexpr int BT = 16 * SPL;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int g = lane >> 4, u = lane & 15;
    const int d = a.d;
    const int b0 = blockIdx.y * BT;
    const int nb = min(BT, a.B - b0);

    tk_stage<BT>(a, b0, nb);

    const int xl = u * SPL * (int)sizeof(float);   // LDS byte offset of this lane's samples of column 0
    // Per sample: the lane's sorted list, the score of its last entry once it
    // is full, and whether it is full.  Shared by the workgroup: per sample the
    // highest last-entry score of any full list (as an order-preserving
    // integer, 0 = none), a bound below which no label can still make the
    // sample's top KP; a score equal to it may, by its label, so it passes.
    uint64_t kl[SPL][KP];
    float thr[SPL], thr_sh[SPL];
    bool full[SPL];
#pragma unroll
    for (int e = 0; e < SPL; ++e) {
#pragma unroll
        for (int p = 0; p < KP; ++p) kl[e][p] = 0;
        thr[e] = -INFINITY;
        thr_sh[e] = -INFINITY;
        full[e] = false;
    }
    uint32_t *shared_thr = reinterpret_cast<uint32_t *>(tk_smem + a.thr_off);
    // lmax[bt * TK_LISTS + list]: best score of each list (0 = empty).  The
    // K-th largest of a sample's 32 list bests is also a bound: K distinct
    // labels reach it.
    uint32_t *lmax = shared_thr + BT;
    const int my_list = wave * TK_ROWS + g;

    const int rounds = (a.k + 31) >> 5;
    const int64_t stride = (int64_t)gridDim.x * TK_WAVES * TK_ROWS;
    int64_t l0 = ((int64_t)blockIdx.x * TK_WAVES + wave) * TK_ROWS;
    int r = 0;
    // ring of row data, TK_AHEAD steps of (row group, round) ahead
    TkRaw ring[TK_AHEAD];
    int64_t ll0 = l0;
    int lr = 0;
#pragma unroll
    for (int i = 0; i < TK_AHEAD; ++i) {
        if (ll0 < a.L) tk_load(a, ll0, lr, g, u, ring[i]);
        if (++lr == rounds) {
            lr = 0;
            ll0 += stride;
        }
    }
    float z[SPL];
#pragma unroll
    for (int e = 0; e < SPL; ++e) z[e] = 0.f;
    float zb = 0.f;
    bool more = l0 < a.L;
    int steps = 0;
    while (more) {
#pragma unroll
        for (int i = 0; i < TK_AHEAD; ++i) {
            if (more) {   // uniform
                const TkRaw cur = ring[i];
                if (ll0 < a.L) tk_load(a, ll0, lr, g, u, ring[i]);
                if (++lr == rounds) {
                    lr = 0;
                    ll0 += stride;
                }

                if (r == 0) zb = cur.bias;
                const TkRound rd = tk_prep<SPL>(cur, d, a.idx16);
                const int npairs = min(16, (a.k - 32 * r + 1) >> 1);
                if (npairs == 16)
                    tk_round_full<SPL>(rd, xl, z);
                else
                    tk_round_part<SPL>(rd, xl, npairs, z);

                if (r == rounds - 1) {
                    const int64_t l = l0 + g;
                    const bool valid = l < a.L;
                    ++steps;
                    if ((steps & (steps - 1)) == 0 || (steps & 63) == 0)
                        tk_list_bound<KP, BT>(lmax, shared_thr, a.K, wave, lane);
                    if ((steps & 3) == 0) {
                        // refresh the workgroup's bounds for this lane's samples
#pragma unroll
                        for (int e = 0; e < SPL; ++e)
                            thr_sh[e] = key_score((uint64_t)__hip_atomic_load(shared_thr + u * SPL + e, __ATOMIC_RELAXED,
                                                                              __HIP_MEMORY_SCOPE_WORKGROUP)
                                                  << 32);
                    }
#pragma unroll
                    for (int e = 0; e < SPL; ++e) {
                        const float ze = z[e] + zb;
                        // this lane's rows come in ascending label order, so a
                        // score equal to its own last entry's loses the tie;
                        // NaN never enters
                        const bool hit = valid & (u * SPL + e < nb) & ((ze > thr[e]) | (!full[e] & (ze == ze))) &
                                         (ze >= thr_sh[e]);
                        if (__builtin_amdgcn_ballot_w64(hit) != 0) {
                            if (hit) {
                                list_insert(kl[e], score_key(ze, (uint32_t)l));
                                lmax[(u * SPL + e) * TK_LISTS + my_list] = (uint32_t)(kl[e][0] >> 32);
                                full[e] = kl[e][KP - 1] != 0;
                                if (full[e]) {
                                    thr[e] = key_score(kl[e][KP - 1]);
                                    atomicMax(shared_thr + u * SPL + e, (uint32_t)(kl[e][KP - 1] >> 32));
                                }
                            }
                        }
                        z[e] = 0.f;
                    }
                }
                if (++r == rounds) {
                    r = 0;
                    l0 += stride;
                }
                more = l0 < a.L;
            }
        }
    }

    // merge the workgroup's 32 lists per sample into one
    __syncthreads();   // the X tile is no longer read
    uint64_t *Ls = reinterpret_cast<uint64_t *>(tk_smem);
#pragma unroll
    for (int e = 0; e < SPL; ++e) {
        const int bt = u * SPL + e;
        uint64_t *dst = Ls + ((size_t)bt * TK_LISTS + wave * TK_ROWS + g) * KP;
#pragma unroll
        for (int p = 0; p < KP; ++p) dst[p] = kl[e][p];
    }
    tk_merge_lists<KP, BT>(a, b0, nb);
}

// ---------------------------------------------------------------------------
// k_topk_any: the scan for bf16 values of every fan-in and of the widths whose
// tile holds 64, 32 or 16 samples: NP samples per lane, the fan-in in rounds
// of 32 slots gathered with transposing LDS reads (gather_dev.h), the next two
// rounds in flight.
//
// What bounds it: the LDS gathers and their bank conflicts.  With rows loaded
// by all 16 lanes instead (fan-in 64, width 2048, 1048576 labels, B 128, top
// 5) the scan took 846 us, against 692 with each value loaded once and crossed
// by DPP; lists that also take the other workgroups' bests as bounds, four waves
// per SIMD and a short merge take it to 572, the VALU busy 65% of the time and
// the LDS 56%, 63% of that bank conflicts.  (The scan it replaced, each lane
// gathering its own samples at two waves per SIMD: 1379.  Fan-in 32, width 768,
// 2812281 labels, B 64: 424 -> 348.)
//
// 1024 threads, four waves per SIMD, while the lists leave the registers for
// them; past 20 keys a lane 512 threads.
//
// The tile comes from an X image prepared once per call, or without the room
// for one (the no-allocation call at its limit) from X.
constexpr int any_threads(int NP, int KP) { return NP * KP <= 20 ? 1024 : 512; }

__device__ __forceinline__ uint32_t row_max_u32(uint32_t v) {
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false));   // row_ror:8
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false));
    v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false));
    return v;
}

// K-th largest of a row's 16 values (equal ones leave together: a lower
// bound still)
__device__ __forceinline__ uint32_t row_kth_u32(uint32_t v, int K) {
    uint32_t m = 0u;
    for (int r = 0; r < K; ++r) {
        m = row_max_u32(v);
        v = v == m ? 0u : v;
    }
    return m;
}

// Bounds of the samples a wave answers for, 16 lanes each: the K-th largest
// of the bests of 16 groups of the workgroup's lists, and of 16 groups of the
// first TK_SHARE workgroups, which publish theirs in a.best (K distinct labels
// reach either).  Not of all workgroups: reading 512 bests per sample cost
// more than the tighter bound saved (1000000 labels of fan-in 7, B 64, top 8:
// 343 us, with 64 of them 172).
// A best read late is only lower, so results don't depend on the order in
// which workgroups run.
template <int BT, int TH>
__device__ __forceinline__ void tk_bounds(const TkArgs &a, const uint32_t *lmax, uint32_t *shared_thr, int b0, int nb,
                                          int wave, int lane) {
    constexpr int LISTS = TH / 16, PER = BT / (TH / 64);
    const int u = lane & 15;
#pragma unroll
    for (int s = 0; s < PER; s += 4) {
        const int at = s + (lane >> 4), bt = wave * PER + at;
        const bool on = at < PER && bt < nb;
        uint32_t v = 0u, w = 0u;
        if (on) {
#pragma unroll
            for (int i = 0; i < LISTS / 16; ++i)
                v = max(v, __hip_atomic_load(lmax + bt * LISTS + 16 * i + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
        }
        const uint32_t own = row_max_u32(v);
        if (on && a.best) {
            uint32_t *row = a.best + (size_t)(b0 + bt) * TK_SHARE;
            if (u == 0 && blockIdx.x < TK_SHARE)
                __hip_atomic_store(row + blockIdx.x, own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int i = 0; i < TK_SHARE / 16; ++i)
                w = max(w, __hip_atomic_load(row + 16 * i + u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        }
        const uint32_t m = max(row_kth_u32(v, a.K), row_kth_u32(w, a.K));
        if (on && u == 0 && m) atomicMax(shared_thr + bt, m);
    }
}

template <int NP, int KP, bool FULL, bool IDX16>
__global__ __launch_bounds__(any_threads(NP, KP)) void k_topk_any(TkArgs a) {
    using namespace gdev;
    extern __shared__ __align__(16) unsigned char st_smem[];
    constexpr int TH = any_threads(NP, KP), NW = TH / 64, LISTS = TH / 16, BT = 16 * NP;
    constexpr uint32_t COL = 32u * NP;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = lane >> 4, q = lane & 15;
    const int d = a.d, k = a.k;
    const int b0 = blockIdx.y * BT, nb = min(BT, a.B - b0);
    const int64_t r0 = blockIdx.x * a.rows_per_wg;
    const uint32_t rows = (uint32_t)min(a.L - r0, a.rows_per_wg);
    const Rsrc rI = make_rsrc(reinterpret_cast<const char *>(a.I) + r0 * k * (IDX16 ? 2 : 4), rows * (uint32_t)k * (IDX16 ? 2u : 4u));
    const Rsrc rW = make_rsrc(static_cast<const uint16_t *>(a.W) + r0 * k, rows * (uint32_t)k * 2u);
    const Rsrc rB = make_rsrc(a.bias ? a.bias + r0 : nullptr, a.bias ? rows * 4u : 0u);

    const int rounds = (k + 31) >> 5;
    constexpr uint32_t step = 4 * NW;
    uint32_t l_cur = 4u * wave, l_nxt = l_cur;
    int rd_cur = 0, rd_nxt = 0;
    auto advance = [&](uint32_t &l, int &rd) {
        if (++rd == rounds) {
            rd = 0;
            l += step;
        }
    };
    auto load = [&](TrRound<FULL> &o, float &bias) {
        const uint32_t l = l_nxt + grp;   // rows past the end read zeros
        tr_load_round<FULL, IDX16>(rI, rW, l, k, rd_nxt, q, o);
        bias = ldf(rB, l * 4u);
        advance(l_nxt, rd_nxt);
    };
    TrRound<FULL> ra, rb;
    float ba, bb;
    load(ra, ba);
    load(rb, bb);

    const uint32_t image = (uint32_t)(d + 1) * COL;
    if (a.xa) {
        stage_image(a.xa + (size_t)blockIdx.y * image, image, wave, lane, NW);
    } else {
        const uint16_t *X = static_cast<const uint16_t *>(a.X) + (int64_t)b0 * d;
        for (int b = 0; b < BT; ++b) {
            const int r = b / NP;
            for (int c = tid; c <= d; c += TH)
                *reinterpret_cast<uint16_t *>(st_smem + (uint32_t)c * COL + 8 * (NP * (r >> 2) + ((b % NP) ^ staged_swz_a(c, NP))) +
                                              2 * (r & 3)) = (b < nb && c < d) ? X[(int64_t)b * d + c] : (uint16_t)0;
        }
    }
    uint32_t *shared_thr = reinterpret_cast<uint32_t *>(st_smem + a.thr_off);
    uint32_t *lmax = shared_thr + BT;
    for (int i = tid; i < BT * (1 + LISTS); i += TH) shared_thr[i] = 0u;
    __syncthreads();

    // accumulator e is sample NP q + (e ^ gx)
    const int gx = grp & (NP - 1);
    const uint32_t pbase = 8u * NP * (q & 3) + 8u * gx;
    const int my_list = wave * 4 + grp;
    uint64_t kl[NP][KP];
    float thr[NP], thr_sh[NP];
    bool full[NP];
    auto smp = [&](int e) { return NP * q + (e ^ gx); };
#pragma unroll
    for (int e = 0; e < NP; ++e) {
#pragma unroll
        for (int p = 0; p < KP; ++p) kl[e][p] = 0;
        thr[e] = -INFINITY;
        thr_sh[e] = smp(e) < nb ? -INFINITY : INFINITY;
        full[e] = false;
    }
    const int kk = a.K - 1;   // the entry whose score bounds this lane's list (K <= KP)
    int steps = 0;
    float z[NP];
#pragma unroll
    for (int e = 0; e < NP; ++e) z[e] = 0.f;

    auto process = [&](const TrRound<FULL> &o, float bias) {
        tr_round<NP, FULL>(o, d, k - 32 * rd_cur, q, pbase, z);
        if (rd_cur == rounds - 1) {
            const uint32_t l = l_cur + grp;
            const bool valid = l < rows;
            ++steps;
            // what is new since the last time halves with every doubling
            const bool refresh = (steps & (steps - 1)) == 0 || (steps & 63) == 0;
            if (refresh) tk_bounds<BT, TH>(a, lmax, shared_thr, b0, nb, wave, lane);
            if (refresh || (steps & 3) == 0) {
#pragma unroll
                for (int e = 0; e < NP; ++e)
                    if (smp(e) < nb)
                        thr_sh[e] = key_score((uint64_t)__hip_atomic_load(shared_thr + smp(e), __ATOMIC_RELAXED,
                                                                          __HIP_MEMORY_SCOPE_WORKGROUP)
                                              << 32);
            }
            // A lane's rows come in ascending label order, so a score equal
            // to its own last entry's loses the tie; one equal to a bound may
            // still win it; NaN never enters.
            float ze[NP];
            bool hit[NP];
            bool any = false;
#pragma unroll
            for (int e = 0; e < NP; ++e) {
                ze[e] = z[e] + bias;
                hit[e] = valid & (ze[e] >= thr_sh[e]) & ((ze[e] > thr[e]) | !full[e]);
                any |= hit[e];
                z[e] = 0.f;
            }
            if (__builtin_amdgcn_ballot_w64(any) != 0) {
#pragma unroll
                for (int e = 0; e < NP; ++e) {
                    if (hit[e]) {
                        list_insert(kl[e], score_key(ze[e], (uint32_t)(r0 + l)));
                        lmax[smp(e) * LISTS + my_list] = (uint32_t)(kl[e][0] >> 32);
                        uint64_t kth = kl[e][KP - 1];
                        if (kk != KP - 1) {
#pragma unroll
                            for (int p = 0; p < KP - 1; ++p) kth = p == kk ? kl[e][p] : kth;
                        }
                        full[e] = kth != 0;
                        if (full[e]) {
                            thr[e] = key_score(kth);
                            atomicMax(shared_thr + smp(e), (uint32_t)(kth >> 32));
                        }
                    }
                }
            }
        }
        advance(l_cur, rd_cur);
    };
    while (l_cur < rows) {
        process(ra, ba);
        load(ra, ba);
        if (l_cur >= rows) break;
        process(rb, bb);
        load(rb, bb);
    }

    __syncthreads();   // the tile is no longer read
    uint64_t *Ls = reinterpret_cast<uint64_t *>(st_smem);
#pragma unroll
    for (int e = 0; e < NP; ++e) {
        uint64_t *dst = Ls + ((size_t)smp(e) * LISTS + my_list) * KP;
#pragma unroll
        for (int p = 0; p < KP; ++p) dst[p] = kl[e][p];
    }
    tk_merge_lists<KP, BT, TH>(a, b0, nb);
}

// block-wide maximum of one key per thread (TK_MERGE_THREADS threads)
__device__ __forceinline__ uint64_t block_max_key(uint64_t x, uint64_t *red) {
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        const uint32_t lo = __shfl_xor((uint32_t)x, s, 64);
        const uint32_t hi = __shfl_xor((uint32_t)(x >> 32), s, 64);
        const uint64_t y = ((uint64_t)hi << 32) | lo;
        x = y > x ? y : x;
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) red[wave] = x;
    __syncthreads();
    uint64_t mx = red[0];
#pragma unroll
    for (int w = 1; w < TK_MERGE_THREADS / 64; ++w) mx = red[w] > mx ? red[w] : mx;
    __syncthreads();
    return mx;
}

template <int KP>
__global__ __launch_bounds__(TK_MERGE_THREADS) void k_topk_merge(const uint64_t *part, int nwg, int K,
                                                                  int32_t *top_lab, float *top_sc,
                                                                  const int32_t *off, const int32_t *lab,
                                                                  uint8_t *rel) {
    __shared__ uint64_t red[TK_MERGE_THREADS / 64];
    __shared__ uint64_t win[16];
    const int b = blockIdx.x, tid = threadIdx.x;
    const uint64_t *pb = part + (size_t)b * nwg * KP;
    uint64_t kl[KP];
#pragma unroll
    for (int p = 0; p < KP; ++p) kl[p] = 0;
    if (tid < nwg) {
#pragma unroll
        for (int p = 0; p < KP; ++p) kl[p] = pb[(size_t)tid * KP + p];
    }
    for (int i = tid + TK_MERGE_THREADS; i < nwg; i += TK_MERGE_THREADS) list_merge(kl, pb + (size_t)i * KP);
    // K rounds: the best head wins and its list moves up by one
    for (int j = 0; j < K; ++j) {
        const uint64_t w = block_max_key(kl[0], red);
        if (w != 0 && kl[0] == w) {
#pragma unroll
            for (int p = 0; p < KP - 1; ++p) kl[p] = kl[p + 1];
            kl[KP - 1] = 0;
        }
        if (tid == 0) win[j] = w;
    }
    __syncthreads();
    if (tid < K) {
        const uint64_t w = win[tid];
        const int32_t l = key_label(w);
        top_lab[(size_t)b * K + tid] = l;
        if (top_sc) top_sc[(size_t)b * K + tid] = w ? key_score(w) : -INFINITY;
        if (rel) {
            uint8_t hit = 0;
            if (l >= 0)
                for (int e = off[b]; e < off[b + 1]; ++e)
                    if (lab[e] == l) {
                        hit = 1;
                        break;
                    }
            rel[(size_t)b * K + tid] = hit;
        }
    }
}

// out[j] = mean over samples of (1/(j+1)) * (relevant among the first j+1)
constexpr int TK_PATK_THREADS = 256;
__global__ __launch_bounds__(TK_PATK_THREADS) void k_patk(const uint8_t *rel, int B, int K, float *out) {
    __shared__ int32_t part[16][TK_PATK_THREADS];
    const int t = threadIdx.x;
    int32_t acc[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = 0;
    for (int b = t; b < B; b += TK_PATK_THREADS) {
        int32_t h = 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            if (j < K) h += rel[(size_t)b * K + j];
            acc[j] += h;
        }
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) part[j][t] = acc[j];
    __syncthreads();
    for (int s = TK_PATK_THREADS / 2; s > 0; s >>= 1) {
        if (t < s)
#pragma unroll
            for (int j = 0; j < 16; ++j) part[j][t] += part[j][t + s];
        __syncthreads();
    }
    if (t < K) out[t] = (float)((double)part[t][0] / ((double)(t + 1) * (double)B));
}

template <int SPL, int KP>
const void *scan_kernel() {
    if constexpr (SPL * KP <= 16)
        return reinterpret_cast<const void *>(&k_topk_scan<SPL, KP>);
    else
        return nullptr;
}
template <int SPL>
const void *pick_kp(int kp) {
    return kp == 1 ? scan_kernel<SPL, 1>() : kp == 4 ? scan_kernel<SPL, 4>() : kp == 8 ? scan_kernel<SPL, 8>()
                                                                                   : scan_kernel<SPL, 16>();
}
const void *pick_spl(int spl, int kp) {
    return spl == 4 ? pick_kp<4>(kp) : spl == 2 ? pick_kp<2>(kp) : pick_kp<1>(kp);
}

// the bf16 scan keeps lists of exactly 1, 3 or 5 entries for the usual P@1,
// P@3 and P@5 (an insert costs one compare and select per entry), and no more
// than 4, 8 or 16 for the others: the lists are what fills the no-allocation
// call's scratch
int list_kp(int topk) { return topk == 1 ? 1 : topk <= 3 ? 3 : topk <= 5 ? topk : topk <= 8 ? 8 : 16; }

template <int NP, int KP>
const void *any_kernel_f(bool full, bool i16) {
    return full ? (i16 ? reinterpret_cast<const void *>(&k_topk_any<NP, KP, true, true>)
                       : reinterpret_cast<const void *>(&k_topk_any<NP, KP, true, false>))
                : (i16 ? reinterpret_cast<const void *>(&k_topk_any<NP, KP, false, true>)
                       : reinterpret_cast<const void *>(&k_topk_any<NP, KP, false, false>));
}
template <int NP>
const void *any_kernel(int kp, bool full, bool i16) {
    switch (kp) {
    case 1: return any_kernel_f<NP, 1>(full, i16);
    case 3: return any_kernel_f<NP, 3>(full, i16);
    case 4: return any_kernel_f<NP, 4>(full, i16);
    case 5: return any_kernel_f<NP, 5>(full, i16);
    case 8: return any_kernel_f<NP, 8>(full, i16);
    default:
        if constexpr (NP <= 2) return any_kernel_f<NP, 16>(full, i16);
        return nullptr;
    }
}
size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

bool topk_shape(const Layer &ly, int B, int topk, TopkPlan *p, bool image) {
    if (topk < 1 || topk > FFSL_MAX_TOPK || B < 1 || B > FFSL_MAX_B) return false;
    if (ly.L >= ((int64_t)1 << 31)) return false;
    const bool bf = ly.vt == FFSL_BF16;
    const int elt = bf ? 2 : 4;
    p->kp = topk == 1 ? 1 : topk <= 4 ? 4 : topk <= 8 ? 8 : 16;
    // list registers per lane: spl * kp keys (fp32 lanes also hold wider gathers)
    const int max_keys = bf ? 32 : 16;
    // the tile, and after it the bounds and the bests of the workgroup's lists
    auto fits = [&](int s) {
        const size_t tile = (size_t)(ly.d + 1) * 16 * s * elt;
        return tile <= TOPK_XS_MAX && align256(tile) + sizeof(uint32_t) * 16 * s * (bf ? 65 : 33) <= TOPK_LDS_MAX;
    };
    int spl = 4;
    while (spl > 1 && (!fits(spl) || spl * p->kp > max_keys || 16 * (spl / 2) >= B)) spl /= 2;
    if ((size_t)(ly.d + 1) * 16 * spl * elt > TOPK_XS_MAX) return false;
    p->spl = spl;
    p->bt = 16 * spl;
    p->tiles = (B + p->bt - 1) / p->bt;
    p->thr_off = (int)align256((size_t)(ly.d + 1) * p->bt * elt);
    p->threads = TK_THREADS;
    if (bf) {
        // lists of exactly 1, 3 or 5 entries for the usual P@1, P@3 and P@5
        p->kp = list_kp(topk);
        const bool full = ly.k % 32 == 0, i16 = ly.idx16 != 0;
        p->scan = spl == 4 ? any_kernel<4>(p->kp, full, i16) : spl == 2 ? any_kernel<2>(p->kp, full, i16)
                                                                        : any_kernel<1>(p->kp, full, i16);
        p->threads = any_threads(spl, p->kp);
    } else {
        p->scan = pick_spl(spl, p->kp);
    }
    if (!p->scan) return false;
    const int lists = p->threads / 16;
    p->lds = std::max((size_t)p->thr_off + sizeof(uint32_t) * p->bt * (1 + lists), (size_t)p->bt * lists * p->kp * 8);
    p->nwg = 0;
    p->part = 0;
    p->rel = align256(sizeof(uint64_t) * (size_t)B * (size_t)ly.num_cu * TOPK_MAX_WG_PER_CU * p->kp);
    p->total = p->rel + align256((size_t)B * topk);
    p->img = bf && image ? p->total : 0;
    if (p->img) p->total += align256((size_t)p->tiles * (ly.d + 1) * p->bt * 2);
    p->best = p->total;
    if (p->img) p->total += align256(sizeof(uint32_t) * (size_t)B * TK_SHARE);
    return true;
}

int topk_grid(const Layer &ly, TopkPlan *p) {
    hipError_t e = hipFuncSetAttribute(p->scan, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p->lds);
    if (e != hipSuccess) return fail(FFSL_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
    int occ = 0;
    e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, p->scan, p->threads, p->lds);
    if (e != hipSuccess) return fail(FFSL_EHIP, "hipOccupancyMaxActiveBlocksPerMultiprocessor: %s",
                                     hipGetErrorString(e));
    occ = std::max(1, std::min(occ, TOPK_MAX_WG_PER_CU));
    const int64_t step = p->threads / 16;   // rows a workgroup takes at a time
    const int64_t need = (ly.L + step - 1) / step;
    int64_t nwg = std::max<int64_t>(1, std::min<int64_t>((int64_t)ly.num_cu * occ, need));
    if (ly.vt == FFSL_BF16) {
        p->rows_per_wg = ((ly.L + nwg - 1) / nwg + step - 1) / step * step;
        nwg = (ly.L + p->rows_per_wg - 1) / p->rows_per_wg;
    }
    p->nwg = (int)nwg;
    return FFSL_OK;
}

int launch_topk(const Layer &ly, const void *X, int B, int topk, int32_t *top_lab, float *top_sc,
                const int32_t *off, const int32_t *lab, float *p_at_k, char *ws, const TopkPlan &p,
                hipStream_t st) {
    TkArgs a{};
    a.X = X;
    a.W = ly.W;
    a.I = ly.I;
    a.idx16 = ly.idx16;
    a.bias = ly.bias;
    a.L = ly.L;
    a.B = B;
    a.d = ly.d;
    a.k = ly.k;
    a.nwg = p.nwg;
    a.thr_off = p.thr_off;
    a.K = topk;
    a.part = reinterpret_cast<uint64_t *>(ws + p.part);
    a.rows_per_wg = p.rows_per_wg;
    int rc;
    if (p.img) {
        StagedPrepArgs pa{};
        pa.X = X;
        pa.B = B;
        pa.d = ly.d;
        pa.xa = reinterpret_cast<unsigned char *>(ws + p.img);
        pa.p.BT = pa.p.BTW = p.bt;
        pa.p.tiles = p.tiles;
        pa.p.cola = p.bt * 2;
        a.best = pa.zero = reinterpret_cast<uint32_t *>(ws + p.best);
        pa.nzero = B * TK_SHARE;
        rc = launch_staged_prep(ly, pa, st);
        if (rc) return rc;
        a.xa = pa.xa;
    }
    uint8_t *rel = p_at_k ? reinterpret_cast<uint8_t *>(ws + p.rel) : nullptr;
    hipLaunchKernelGGL(reinterpret_cast<void (*)(TkArgs)>(const_cast<void *>(p.scan)), dim3(p.nwg, p.tiles),
                       dim3(p.threads), p.lds, st, a);
    rc = check_launch("k_topk_scan");
    if (rc) return rc;
    switch (p.kp) {
    case 1: hipLaunchKernelGGL(k_topk_merge<1>, dim3(B), dim3(TK_MERGE_THREADS), 0, st, a.part, p.nwg, topk,
                               top_lab, top_sc, off, lab, rel); break;
    case 3: hipLaunchKernelGGL(k_topk_merge<3>, dim3(B), dim3(TK_MERGE_THREADS), 0, st, a.part, p.nwg, topk,
                               top_lab, top_sc, off, lab, rel); break;
    case 4: hipLaunchKernelGGL(k_topk_merge<4>, dim3(B), dim3(TK_MERGE_THREADS), 0, st, a.part, p.nwg, topk,
                               top_lab, top_sc, off, lab, rel); break;
    case 5: hipLaunchKernelGGL(k_topk_merge<5>, dim3(B), dim3(TK_MERGE_THREADS), 0, st, a.part, p.nwg, topk,
                               top_lab, top_sc, off, lab, rel); break;
    case 8: hipLaunchKernelGGL(k_topk_merge<8>, dim3(B), dim3(TK_MERGE_THREADS), 0, st, a.part, p.nwg, topk,
                               top_lab, top_sc, off, lab, rel); break;
    default: hipLaunchKernelGGL(k_topk_merge<16>, dim3(B), dim3(TK_MERGE_THREADS), 0, st, a.part, p.nwg, topk,
                                top_lab, top_sc, off, lab, rel); break;
    }
    rc = check_launch("k_topk_merge");
    if (rc || !p_at_k) return rc;
    hipLaunchKernelGGL(k_patk, dim3(1), dim3(TK_PATK_THREADS), 0, st, rel, B, topk, p_at_k);
    return check_launch("k_patk");
}

}  // namespace ffsl

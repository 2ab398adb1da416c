// Host side of libgdn: argument validation, workspace layout and caching,
// kernel launches, and the extern "C" entry points declared in gdn.h.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <unordered_map>
#include <utility>
#include <vector>

#include "gdn.h"
#include "gdn_frame.h"
#include "gdn_kernels.h"

namespace {

using gdn::kChunk;
using gdn::kGateRec;

struct WsLayout {
    size_t er, gf, W, Ut, Hs, Us, Nf, PsiT, lgam, HgT, total;
};

size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

int num_chunks(int T) { return (T + kChunk - 1) / kChunk; }

// Chunks per scan group.  bf16: a single group (one sequential scan per
// (b, h)) whenever the (b, h) streams give at least 64 column-tile workgroups or
// the sequence has at most 64 chunks.  fp32, and bf16 with fewer streams: a single
// group when the sequence is short or when the streams alone fill the chip;
// otherwise about sqrt(NC) chunks per group, which balances the group-parallel
// passes (two passes over G chunks) against the sequential scan over NC / G groups.
// Measured (us a call, single -> best grouped; bf16, D = 128 unless said): T = 3520,
// H = 16 59.4 -> 68.1; T = 10560, H = 16 172.5 -> 185.3; T = 42240, H = 32 1026 ->
// 1480; T = 10560, 80 heads of D = 64 303 -> 428; T = 10560, H = 4 124.8 -> 66.9
// (68.6 at this rule's G = 13).  The line lies where the passes before the present
// ones crossed; with the present ones H = 8 at T = 10560 takes 135.8 single and
// 102.4 at G = 26, and fp32 H = 16 641 single and 736 at this rule's G = 13.  It is
// part of the interface (gdn_scan_group_size, workspace sizes) and stays.
int auto_group(int NC, long long BH, int Dv, bool bf16) {
    if (NC <= 64 || BH * (Dv / 16) >= (bf16 ? 64 : 512)) return NC;
    int G = (int)(__builtin_sqrt((double)NC) + 0.5);
    return G < 2 ? 2 : G;
}

int resolve_group(int NC, long long BH, int Dv, int group, bool bf16) {
    if (group <= 0) group = auto_group(NC, BH, Dv, bf16);
    return group > NC ? NC : group;
}

// fp32, and bf16 with several scan groups: the output takes the queries unscaled
// (the kernels' RAW variant).
bool raw_queries(size_t esz, int NG) { return esz == 4 || NG > 1; }

WsLayout ws_layout(int B, int H, int T, int Dk, int Dv, size_t esz, int G) {
    const int NC = num_chunks(T);
    const int NG = (NC + G - 1) / G;
    const size_t bh = (size_t)B * H;
    const size_t nch = bh * NC;
    const size_t ngr = NG > 1 ? bh * NG : 0;
    WsLayout L;
    size_t off = 0;
    L.er = off;   off = align256(off + nch * kChunk * 8);
    L.gf = off;   off = align256(off + nch * kGateRec * 4);
    L.W = off;    off = align256(off + nch * kChunk * Dk * esz);
    L.Ut = off;   off = align256(off + nch * Dv * kChunk * esz);
    // These regions hold the chunk's queries (C x Dk) and masked scores (C x C).
    // In fp32 and with several groups they keep the sizes of the per-chunk state
    // (Dv x Dk) and pseudo-values (Dv x C) that an output kernel of its own once
    // read there, and er those of its fp64 log decays (a single bf16 scan has no
    // use for er): a caller's workspace is sized the same as ever.
    const bool fused = esz == 2 && NG == 1;
    L.Hs = off;   off = align256(off + nch * (fused ? kChunk : Dv) * Dk * esz);
    L.Us = off;   off = align256(off + nch * (fused ? kChunk : Dv) * kChunk * esz);
    L.Nf = off;   off = align256(off + ngr * Dk * Dk * esz);
    L.PsiT = off; off = align256(off + ngr * Dv * Dk * 4);
    L.lgam = off; off = align256(off + ngr * 8);
    L.HgT = off;  off = align256(off + ngr * Dv * Dk * 4);
    L.total = off;
    return L;
}

// A single-group call whose chunk records (W, U~, Q~, P: 56 KB a chunk and head at
// D = 128) outgrow the 256 MB memory-side cache is run in slabs of consecutive
// chunks that do not: the WY kernel and the scan of one slab, then the next
// one's in the same records, the state carried in fp32 through the workspace
// (the records past the first slab are free).  The scan then reads the records
// from that cache and not from HBM, which takes them in and out at half the
// speed the scan needs.  Same kernels, same order of every sum: same bits.
// Measured (us a call, one pass -> slabs): T = 12288, H = 16 271 -> 207, T = 16384
// 388 -> 269, T = 42240, H = 32 1231 -> 1008, 80 heads of D = 64 at T = 10560
// 358 -> 303.  Slabs of 112 MB: 104 to 128 are equal, 88 and 160 up to 5 and 14 %
// slower, 40 no gain (each slab's launches and ring fill cost some 8 us).
// Two slabs against one pass over the records' size: 16 heads of D = 128 at 119 MB
// 145.7 -> 151.8, 127 MB 158.3 -> 158.0, 134 MB 171.3 -> 165.2, 140 MB 185.8 ->
// 172.3, 144.4 MB (T = 10560) 196.1 -> 177.5; 32 heads at 114 MB 98.9 -> 109.3, 128
// MB 116.9 -> 116.3, 136 MB 132.5 -> 123.0; 64 heads at 126 MB 98.6 -> 103.4, 140 MB
// 113.6 -> 112.1; 80 heads of D = 64 at 132 MB 100.7 -> 103.1, 142 MB 107.6 -> 106.4;
// 16 of D = 64 at 124 MB 170.6 -> 177.5, 136 MB 191.0 -> 192.1, 146 MB 218.3 ->
// 206.2; 16 of 128 x 64 at 121 MB 160.9 -> 164.4, 133 MB 182.3 -> 177.4.  The
// curves cross between 127 and 138 MB; with the line at 132 MB none of these shapes
// loses more than some 3 % near it.
// Fewer than 16 chunks to a slab (more than 128 heads of D = 128, 224 of D = 64)
// would pay more for the carried state than it saves (200 heads of D = 128, 16
// chunks 168.3 -> 171.1, 32 chunks 321.8 -> 341.6); the fp32 path is bound by its
// MFMAs and gains nothing.
constexpr long long kSlabBytes = 112LL << 20, kSlabsFrom = 132LL << 20;

// Chunks per slab (NC: one pass).  More than 132 MB with 16 chunks or more to 112 MB
// are 19 chunks or more, so the first slab leaves NC / 2 >= 9 chunks of W records
// for the carried state, which takes Dv / 32 <= 4, twice.
int slab_chunks(int B, int H, int NC, int NG, int Dk, int Dv, size_t esz) {
    if (esz != 2 || NG > 1) return NC;
    const long long col = 2LL * kChunk * (2 * Dk + Dv + kChunk) * B * H, most = kSlabBytes / col;
    if (col * NC <= kSlabsFrom || most < 16) return NC;
    const long long n = (NC + most - 1) / most;
    return (int)((NC + n - 1) / n);
}

// Bytes each workspace region must span for the kernels that use it, from the
// kernels' index expressions evaluated at their largest indices (chunk index
// cidx = B H NC - 1, group index gidx = B H NG - 1, lane 63, last fragment):
// the highest element offset touched, plus the element's width.  0 if no
// kernel of the path uses the region.
struct WsNeeds {
    size_t er, gf, W, Ut, Hs, Us, Nf, PsiT, lgam, HgT;
};

WsNeeds ws_needs(int B, int H, int T, int Dk, int Dv, size_t esz, int G) {
    const size_t NC = (size_t)num_chunks(T), NG = (NC + G - 1) / G;
    const size_t cmax = (size_t)B * H * NC - 1;             // last chunk record
    const size_t gmax = (size_t)B * H * NG - 1;             // last group record
    const size_t KB = (size_t)Dk / 32, NJ = (size_t)Dv / 16;
    WsNeeds n{};
    // WY kernel (fp32, and bf16 with several groups): er[cidx * 64 + r]
    if (raw_queries(esz, (int)NG)) n.er = (cmax * kChunk + kChunk) * 4;
    // WY kernel: gf[cidx * 68 + l] and the fp64 g_C at gf + cidx * 68 + 64 (the
    // scan copies gf[cidx * 68 + 4 l .. + 3], l < 17)
    n.gf = (cmax * kGateRec + kGateRec) * 4;
    // -W fragment ((wv * 4 + st) * 2 + kb) * 512 + l * 8, 8 elements
    n.W = (cmax * kChunk * Dk + ((((size_t)Dk / 64 - 1) * 4 + 3) * 2 + 1) * 512 + 63 * 8 + 8) * esz;
    // in slabs: the carried states, [B H][Dk][Dv] fp32 twice, behind the first slab's records
    const size_t SC = slab_chunks(B, H, (int)NC, (int)NG, Dk, Dv, esz);
    if (SC < NC) {
        const size_t carry = (size_t)B * H * (SC * kChunk * Dk * esz + 2 * (size_t)Dk * Dv * 4);
        if (carry > n.W) n.W = carry;
    }
    // U~t quad (4 jt + st) * 256 + l * 4, 4 elements
    n.Ut = (cmax * Dv * kChunk + (4 * (NJ - 1) + 3) * 256 + 63 * 4 + 4) * esz;
    // WY: Qf (rt * KB + kb) * 512 + l * 8 and Pf (rt * 2 + m) * 512 + l * 8
    n.Hs = (cmax * kChunk * Dk + (3 * KB + KB - 1) * 512 + 63 * 8 + 8) * esz;
    n.Us = (cmax * kChunk * kChunk + (3 * 2 + 1) * 512 + 63 * 8 + 8) * esz;
    if (NG > 1) {
        // group transfer: N fragments ((v * 4 + t) * (Dk / 32) + kb) * 512 + l * 8,
        // Psi^T[(gidx * Dv + column) * Dk + row], log Gamma[gidx]; group scan: H^T like Psi^T
        n.Nf = (gmax * Dk * Dk + ((((size_t)Dk / 64 - 1) * 4 + 3) * KB + KB - 1) * 512 + 63 * 8 + 8) * esz;
        n.PsiT = ((gmax * Dv + Dv - 1) * Dk + Dk) * 4;
        n.lgam = (gmax + 1) * 8;
        n.HgT = ((gmax * Dv + Dv - 1) * Dk + Dk) * 4;
    }
    return n;
}

bool shape_ok(int B, int H, int T) {
    if (B < 1 || H < 1 || T < 1) return false;
    // a limit of the interface, from when B*H was a grid dimension (the records of a
    // call with more than 2^31 chunk and head pairs would not fit the memory)
    if ((long long)B * H > 65535) return false;
    return true;
}

bool dims_ok(int Dk, int Dv, int chunk) {
    return (Dk == 64 || Dk == 128) && (Dv == 64 || Dv == 128) && chunk == kChunk;
}

bool misaligned(const void *p) { return p && ((uintptr_t)p & 15u); }

struct Range {
    uintptr_t lo, hi;
    bool valid() const { return lo != 0; }
    bool overlaps(const Range &o) const { return valid() && o.valid() && lo < o.hi && o.lo < hi; }
};
Range range(const void *p, size_t bytes) { return Range{(uintptr_t)p, (uintptr_t)p + bytes}; }

int validate(const void *q, const void *k, const void *v, const float *alpha, const float *beta,
             const float *state_in, const void *out, const float *state_out, int B, int H, int T,
             int Dk, int Dv, int chunk, size_t esz) {
    if (!q || !k || !v || !alpha || !beta || !out) return GDN_ERR_NULL;
    if (!shape_ok(B, H, T)) return GDN_ERR_SHAPE;
    if (!dims_ok(Dk, Dv, chunk)) return GDN_ERR_UNSUPPORTED;
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(alpha) || misaligned(beta) ||
        misaligned(state_in) || misaligned(out) || misaligned(state_out))
        return GDN_ERR_ALIGN;
    const size_t ntok = (size_t)B * T * H;
    const Range rq = range(q, ntok * Dk * esz), rk = range(k, ntok * Dk * esz),
                rv = range(v, ntok * Dv * esz), ra = range(alpha, ntok * 4), rb = range(beta, ntok * 4),
                ro = range(out, ntok * Dv * esz);
    const size_t sbytes = (size_t)B * H * Dk * Dv * 4;
    const Range rsi = range(state_in, sbytes), rso = range(state_out, sbytes);
    const Range ins[] = {rq, rk, rv, ra, rb, rsi};
    for (const Range &r : ins)
        if (ro.overlaps(r)) return GDN_ERR_ALIAS;
    if (rso.valid()) {
        for (int i = 0; i < 5; ++i)
            if (rso.overlaps(ins[i])) return GDN_ERR_ALIAS;
        if (rso.overlaps(ro)) return GDN_ERR_ALIAS;
        if (rsi.valid() && rso.overlaps(rsi) && rso.lo != rsi.lo) return GDN_ERR_ALIAS;
    }
    return GDN_OK;
}

template <class E>
gdn::Params<E> make_params(const void *q, const void *k, const void *v, const float *alpha,
                           const float *beta, const float *state_in, void *out, float *state_out,
                           int B, int H, int T, int Dk, int Dv, int G, void *ws) {
    gdn::Params<E> p;
    p.q = (const E *)q;
    p.k = (const E *)k;
    p.v = (const E *)v;
    p.alpha = alpha;
    p.beta = beta;
    p.state_in = state_in;
    p.out = (E *)out;
    p.state_out = state_out;
    p.B = B;
    p.H = H;
    p.T = T;
    p.NC = num_chunks(T);
    p.c0 = 0;
    p.G = G;
    p.NG = (p.NC + G - 1) / G;
    const WsLayout L = ws_layout(B, H, T, Dk, Dv, sizeof(E), G);
    unsigned char *base = (unsigned char *)ws;
    p.er = (float *)(base + L.er);
    p.gf = (float *)(base + L.gf);
    p.W = (E *)(base + L.W);
    p.Ut = (E *)(base + L.Ut);
    p.Qf = (E *)(base + L.Hs);
    p.Pf = (E *)(base + L.Us);
    p.Nf = (E *)(base + L.Nf);
    p.PsiT = (float *)(base + L.PsiT);
    p.lgam = (double *)(base + L.lgam);
    p.HgT = (float *)(base + L.HgT);
    return p;
}

// Launch one kernel whose only argument is a parameter struct; returns the
// launch's own status (the thread's pending HIP error is neither read nor
// cleared, so an error the caller left pending is not reported as this call's).
template <class P>
hipError_t launch(const void *fn, dim3 grid, dim3 block, size_t lds, hipStream_t s, const P &p) {
    P copy = p;
    void *args[] = {&copy};
    return hipLaunchKernel(fn, grid, block, args, lds, s);
}

constexpr int kStages = 4;  // WY transform, group transfers, group scan, chunk states with output

// Stage timing (measurement aid): every stage that launches is enqueued `reps`
// times back to back between the events ev[2 s] and ev[2 s + 1]; collect() waits
// for them and adds a launch's mean duration to ms[s] (a call in slabs: once each).
struct StageTiming {
    hipEvent_t ev[2 * kStages];
    bool ran[kStages];
    float ms[kStages];
    int reps;
    hipError_t collect() {
        hipError_t e = hipSuccess;
        for (int i = 0; i < kStages && e == hipSuccess; ++i) {
            if (!ran[i]) continue;
            float t = 0.f;
            e = hipEventSynchronize(ev[2 * i + 1]);
            if (e == hipSuccess) e = hipEventElapsedTime(&t, ev[2 * i], ev[2 * i + 1]);
            ms[i] += t / reps;
        }
        return e;
    }
};

template <class E, int DK, int DV, bool RAW>
hipError_t launch_path(const gdn::Params<E> &p, hipStream_t s, StageTiming *tm) {
    constexpr int NOW = 4;                       // output waves
    // Two column tiles per workgroup once one each would be more workgroups than
    // CUs: the pair reads the chunk operands once, and a second round of
    // workgroups or a shared CU costs more than the longer step (us a call, one tile
    // -> two: T = 3520 with 264 tiles of D = 128 115 -> 88, 384 tiles 146 -> 119; T =
    // 10560 with 272 and 320 tiles of D = 64 340 -> 264 and 366 -> 290; 416 tiles in
    // groups 75 -> 68).  Up to one workgroup per CU one tile is faster (T = 3520 with
    // 128 and 256 tiles 59.5 -> 71.0 and 76.4 -> 85.9, T = 42240 with 256 1018 ->
    // 1134, 256 tiles of D = 64 263 -> 269, 208 in groups 52.7 -> 55.6), in fp32
    // always (its two-tile step has no registers for it).
    const bool wide = sizeof(E) == 2 && (long long)p.B * p.H * p.NG * (DV / 16) > 256;
    constexpr int CTW = sizeof(E) == 2 ? 2 : 1;
    using L1 = gdn::ScanLds<E, DK, 1, NOW>;
    using L2 = gdn::ScanLds<E, DK, CTW, NOW>;
    using LT = gdn::ScanLds<E, DK, 2, 0>;        // group transfers
    const void *scan1 = (const void *)gdn::gdn_chunkscan_kernel<E, DK, DV, gdn::SCAN_STATES, 1, NOW, RAW>;
    const void *scan2 = (const void *)gdn::gdn_chunkscan_kernel<E, DK, DV, gdn::SCAN_STATES, CTW, NOW, RAW>;
    const void *scant = (const void *)gdn::gdn_chunkscan_kernel<E, DK, DV, gdn::SCAN_TRANS, 2, 0, true>;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    const size_t lds1 = gdn::WyLds<E, DK, DV>::bytes;
    std::call_once(attr_once, [&] {
        const struct {
            const void *fn;
            size_t bytes;
        } dyn[] = {
            {(const void *)gdn::gdn_wy_kernel<E, DK, DV, RAW>, lds1},
            {scan1, L1::bytes},
            {scan2, L2::bytes},
            {scant, LT::bytes},
        };
        for (const auto &d : dyn) {
            const hipError_t e =
                hipFuncSetAttribute(d.fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)d.bytes);
            if (e != hipSuccess && attr_err == hipSuccess) attr_err = e;
        }
    });
    if (attr_err != hipSuccess) return attr_err;
    const unsigned BH = (unsigned)(p.B * p.H);
    // workgroup counts: column blocks x 8 x ceil(units / 8) (see the XCD placement)
    auto groups = [](unsigned nblocks, unsigned units) { return nblocks * 8u * ((units + 7u) / 8u); };
    auto stage = [&](int i) -> hipError_t {
        switch (i) {
        case 0:
            return launch((const void *)gdn::gdn_wy_kernel<E, DK, DV, RAW>, dim3(p.NC * BH), dim3(64 * gdn::kWyWaves),
                          lds1, s, p);
        case 1:
            return launch(scant, dim3(groups((DK + DV) / 32, BH * p.NG)), dim3(gdn::scan_threads<0>()), LT::bytes, s, p);
        case 2:
            return launch((const void *)gdn::gdn_groupscan_kernel<E, DK, DV>, dim3(groups(DV / 16, BH)),
                          dim3(64 * gdn::kScanSplit), 0, s, p);
        default:
            if (wide)
                return launch(scan2, dim3(groups(DV / (16 * CTW), BH * p.NG)), dim3(gdn::scan_threads<NOW>()), L2::bytes, s, p);
            return launch(scan1, dim3(groups(DV / 16, BH * p.NG)), dim3(gdn::scan_threads<NOW>()), L1::bytes, s, p);
        }
    };
    hipError_t er = hipSuccess;
    for (int i = 0; i < kStages && er == hipSuccess; ++i) {
        const bool runs = (i == 1 || i == 2) ? p.NG > 1 : true;
        if (tm) tm->ran[i] = runs;
        if (!runs) continue;
        if (!tm) {
            er = stage(i);
            continue;
        }
        er = hipEventRecord(tm->ev[2 * i], s);
        for (int r = 0; r < tm->reps && er == hipSuccess; ++r) er = stage(i);
        if (er == hipSuccess) er = hipEventRecord(tm->ev[2 * i + 1], s);
    }
    return er;
}

template <class E, bool RAW>
hipError_t dispatch_raw(const gdn::Params<E> &p, int Dk, int Dv, hipStream_t s, StageTiming *tm) {
    if (Dk == 128 && Dv == 128) return launch_path<E, 128, 128, RAW>(p, s, tm);
    if (Dk == 64 && Dv == 64) return launch_path<E, 64, 64, RAW>(p, s, tm);
    if (Dk == 128 && Dv == 64) return launch_path<E, 128, 64, RAW>(p, s, tm);
    return launch_path<E, 64, 128, RAW>(p, s, tm);
}

template <class E>
hipError_t dispatch(const gdn::Params<E> &p, int Dk, int Dv, hipStream_t s, StageTiming *tm) {
    if constexpr (sizeof(E) == 2)
        if (!raw_queries(sizeof(E), p.NG)) return dispatch_raw<E, false>(p, Dk, Dv, s, tm);
    return dispatch_raw<E, true>(p, Dk, Dv, s, tm);
}

// The whole call.  The carried state alternates between two buffers, so a slab
// whose stages are timed over several launches finds its state as it was.
template <class E>
hipError_t run_slabs(const gdn::Params<E> &p, int Dk, int Dv, hipStream_t s, StageTiming *tm) {
    const int SC = slab_chunks(p.B, p.H, p.NC, p.NG, Dk, Dv, sizeof(E));
    if (SC >= p.NC) {
        const hipError_t e = dispatch(p, Dk, Dv, s, tm);
        return tm && e == hipSuccess ? tm->collect() : e;
    }
    float *carry = (float *)(p.W + (size_t)p.B * p.H * SC * kChunk * Dk);
    float *other = carry + (size_t)p.B * p.H * Dk * Dv;
    hipError_t e = hipSuccess;
    for (int c0 = 0; c0 < p.NC && e == hipSuccess; c0 += SC) {
        gdn::Params<E> r = p;
        r.c0 = c0;
        r.NC = r.G = p.NC - c0 < SC ? p.NC - c0 : SC;
        if (c0) r.state_in = other;
        if (c0 + SC < p.NC) r.state_out = carry;
        e = dispatch(r, Dk, Dv, s, tm);
        if (tm && e == hipSuccess) e = tm->collect();
        std::swap(carry, other);
    }
    return e;
}

int run(const void *q, const void *k, const void *v, const float *alpha, const float *beta,
        const float *state_in, void *out, float *state_out, int B, int H, int T, int Dk, int Dv,
        int chunk, bool bf16, int group, void *ws, size_t ws_bytes, void *stream, StageTiming *tm) {
    const size_t esz = bf16 ? 2 : 4;
    int st = validate(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk, esz);
    if (st != GDN_OK) return st;
    const int G = resolve_group(num_chunks(T), (long long)B * H, Dv, group, bf16);
    if (!ws || ((uintptr_t)ws & 255u) || ws_bytes < ws_layout(B, H, T, Dk, Dv, esz, G).total)
        return GDN_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    hipError_t e;
    if (bf16) {
        e = run_slabs(make_params<uint16_t>(q, k, v, alpha, beta, state_in, out, state_out, B, H, T,
                                           Dk, Dv, G, ws),
                     Dk, Dv, s, tm);
    } else {
        e = run_slabs(make_params<float>(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk,
                                        Dv, G, ws),
                     Dk, Dv, s, tm);
    }
    return e == hipSuccess ? GDN_OK : GDN_ERR_HIP;
}

// Library-cached workspace, one buffer per device, grown on demand.
std::mutex g_ws_mu;
std::unordered_map<int, std::pair<void *, size_t>> g_ws;

int cached_workspace(size_t need, void **ws) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return GDN_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_ws_mu);
    auto &slot = g_ws[dev];
    if (slot.second < need) {
        if (slot.first) {
            if (hipDeviceSynchronize() != hipSuccess) return GDN_ERR_HIP;
            if (hipFree(slot.first) != hipSuccess) return GDN_ERR_HIP;
            slot = {nullptr, 0};
        }
        void *ptr = nullptr;
        if (hipMalloc(&ptr, need) != hipSuccess) return GDN_ERR_HIP;
        slot = {ptr, need};
    }
    *ws = slot.first;
    return GDN_OK;
}

int run_cached(const void *q, const void *k, const void *v, const float *alpha, const float *beta,
               const float *state_in, void *out, float *state_out, int B, int H, int T, int Dk,
               int Dv, int chunk, bool bf16, void *stream) {
    const size_t esz = bf16 ? 2 : 4;
    int st = validate(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk, esz);
    if (st != GDN_OK) return st;
    const size_t need =
        ws_layout(B, H, T, Dk, Dv, esz, resolve_group(num_chunks(T), (long long)B * H, Dv, 0, bf16)).total;
    void *ws = nullptr;
    st = cached_workspace(need, &ws);
    if (st != GDN_OK) return st;
    return run(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk, bf16, 0, ws,
               need, stream, nullptr);
}

// Allocation-free path (gdn_chunk_forward_noalloc): the workspace is a
// file-scope device array, one copy per GPU.  In host code `scratch` names a
// host-side stand-in, not a device address; the address of each GPU's copy
// comes from hipGetSymbolAddress and is kept per device.
static __device__ __align__(256) unsigned char scratch[GDN_NOALLOC_MAX_WORKSPACE];

std::mutex g_scratch_mu;
std::unordered_map<int, void *> g_scratch;  // device -> its copy of `scratch`

int scratch_address(void **ptr) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return GDN_ERR_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    auto it = g_scratch.find(dev);
    if (it == g_scratch.end()) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return GDN_ERR_HIP;
        it = g_scratch.emplace(dev, p).first;
    }
    *ptr = it->second;
    return GDN_OK;
}

int run_noalloc(const void *q, const void *k, const void *v, const float *alpha, const float *beta,
                const float *state_in, void *out, float *state_out, int B, int H, int T, int Dk, int Dv,
                int chunk, void *stream) {
    int st = validate(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk, 2);
    if (st != GDN_OK) return st;
    const size_t need =
        ws_layout(B, H, T, Dk, Dv, 2, resolve_group(num_chunks(T), (long long)B * H, Dv, 0, true)).total;
    if (need > GDN_NOALLOC_MAX_WORKSPACE) return GDN_ERR_WORKSPACE;
    void *ws = nullptr;
    st = scratch_address(&ws);
    if (st != GDN_OK) return st;
    return run(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk, true, 0, ws,
               GDN_NOALLOC_MAX_WORKSPACE, stream, nullptr);
}

// ---------------------------------------------------------------------------
// Frame-wise path (gdn_frame_forward*): frame summaries, their reduction over
// token splits, the scan over frames, and the output; optionally with the
// normalizer state (gdn_frame_forward_norm*) and in the bidirectional form
// (gdn_frame_forward_bidir*).

struct FrameArgs {
    const void *q, *k, *v;
    const float *alpha, *beta, *state_in, *z_in;
    void *out;
    float *state_out, *z_out;
    int B, H, F, N, Dk, Dv;
    float key_scale, eps;
    bool bf16, norm, bidir;
    // the fused operator (gdn_frame_forward_fused*): q and k are the raw
    // projections; the remaining fields are its prologue and epilogue inputs
    bool fused;
    const void *gate, *w_o;
    const float *gain_q, *gain_k, *rope_freq;
    const int *rope_axis;
    float rms_eps;
    int lat_w, t0;
};

struct FrameWs {
    size_t PG, PA, Gf, Af, Hf, Hb, PGz, Gzf, FQ, FKT, FKH, total;
};

int frame_blocks(int N) { return (N + 63) / 64; }

// Token splits per frame: a split is a whole number of 64-token blocks, and
// the library's choice (token_splits <= 0) is the largest count that keeps the
// summary workgroups (one per split) within one per CU (256), at least 1.
int frame_splits(long long units, int N, int token_splits) {
    const int nb = frame_blocks(N);
    int ns = token_splits;
    if (ns <= 0) ns = (int)(256 / units);
    if (ns > nb) ns = nb;
    if (ns < 1) ns = 1;
    const int per = (nb + ns - 1) / ns;   // blocks per split
    return (nb + per - 1) / per;          // no empty split
}

// One layout for every variant: the A tiles, the state fragments and the
// backward histories have room for the normalizer's extra 16-column tile; the
// histories are used by the bidirectional form only, the unrotated-key Gram
// fragments and their partials by the fused operator only.  The fused
// operator in fp32 also keeps its key features and its rotation table (ntok_feat =
// its B F N H token rows; 0 otherwise): the table, F + max(latent rows, columns)
// <= F + N rows of Dk floats, fits the first of these regions (2 ntok_feat rows).
// That region and the unused space at the end once held the query features and
// the gated readout; the total stays, so a workspace is sized the same as ever.
FrameWs frame_ws_layout(int B, int H, int F, int Dk, int Dv, size_t esz, int NS, size_t ntok_feat = 0) {
    const size_t bhf = (size_t)B * H * F;
    const size_t DVn = (size_t)Dv + 16;
    FrameWs L;
    size_t off = 0;
    // partial sums only with several token splits
    const size_t np = NS > 1 ? (size_t)NS : 0;
    L.PG = off; off = align256(off + bhf * np * Dk * Dk * 4);
    L.PA = off; off = align256(off + bhf * np * Dk * DVn * 4);
    L.Gf = off; off = align256(off + bhf * Dk * Dk * esz);
    L.Af = off; off = align256(off + bhf * Dk * DVn * 4);
    L.Hf = off; off = align256(off + bhf * Dk * DVn * esz);
    L.Hb = off; off = align256(off + bhf * Dk * DVn * 4);
    L.PGz = off; off = align256(off + bhf * np * Dk * Dk * 4);
    L.Gzf = off; off = align256(off + bhf * Dk * Dk * esz);
    L.FQ = off;  off = align256(align256(off + ntok_feat * Dk * 4) + ntok_feat * Dk * 4);
    L.FKT = off; off = align256(off + ntok_feat * Dk * 4);
    L.FKH = off; off = align256(off + ntok_feat * Dk * 4);
    off = align256(off + ntok_feat * Dv * 4);
    L.total = off;
    return L;
}

// Token rows whose features the fp32 fused operator keeps in the workspace.
size_t frame_feat_rows(bool fused, bool bf16, int B, int H, int F, int N) {
    return (fused && !bf16) ? (size_t)B * H * F * N : 0;
}

// Output workgroups per (frame, head): about `wgs` workgroups in all, each a
// run of whole 16-token tiles, none empty.
void frame_out_split(long long units, int N, int wgs, int &OB, int &tpw) {
    const int ntf = (N + 15) / 16;
    long long ob = (wgs + units - 1) / units;
    if (ob > ntf) ob = ntf;
    tpw = (int)((ntf + ob - 1) / ob);
    OB = (ntf + tpw - 1) / tpw;
}

bool frame_shape_ok(int B, int H, int F, int N) {
    if (B < 1 || H < 1 || F < 1 || N < 1) return false;
    const long long bh = (long long)B * H;
    if (bh > 65535) return false;
    // token indices (and a split's end, up to 64 * F past the last token) fit in int
    if ((long long)F * N + 64LL * F + N > 0x7fffffffLL) return false;
    // grid sizes of the summary and output kernels stay below 2^31
    const long long units = bh * F;
    if (4LL * frame_blocks(N) * units > 0x7fffffffLL) return false;
    if (8LL * ((N + 15) / 16) * ((units + 7) / 8) > 0x7fffffffLL) return false;
    return true;
}

bool frame_dims_ok(int Dk, int Dv) { return (Dk == 64 || Dk == 128) && (Dv == 64 || Dv == 128); }

int frame_validate(const FrameArgs &a) {
    if (!a.q || !a.k || !a.v || !a.alpha || !a.beta || !a.out) return GDN_ERR_NULL;
    if (!frame_shape_ok(a.B, a.H, a.F, a.N)) return GDN_ERR_SHAPE;
    if (!frame_dims_ok(a.Dk, a.Dv)) return GDN_ERR_UNSUPPORTED;
    if (misaligned(a.q) || misaligned(a.k) || misaligned(a.v) || misaligned(a.alpha) || misaligned(a.beta) ||
        misaligned(a.state_in) || misaligned(a.out) || misaligned(a.state_out) ||
        (a.norm && (misaligned(a.z_in) || misaligned(a.z_out))))
        return GDN_ERR_ALIGN;
    const size_t esz = a.bf16 ? 2 : 4;
    const size_t ntok = (size_t)a.B * a.F * a.N * a.H;
    const Range rq = range(a.q, ntok * a.Dk * esz), rk = range(a.k, ntok * a.Dk * esz),
                rv = range(a.v, ntok * a.Dv * esz), ra = range(a.alpha, (size_t)a.B * a.F * a.H * 4),
                rb = range(a.beta, ntok * 4), ro = range(a.out, ntok * a.Dv * esz);
    const size_t sbytes = (size_t)a.B * a.H * a.Dk * a.Dv * 4, zbytes = (size_t)a.B * a.H * a.Dk * 4;
    const Range rsi = range(a.state_in, sbytes), rso = range(a.state_out, sbytes);
    const Range rzi = range(a.norm ? a.z_in : nullptr, zbytes), rzo = range(a.norm ? a.z_out : nullptr, zbytes);
    // outputs may not overlap the inputs or each other; a state may be updated
    // in place (the same buffer in and out)
    const Range ins[] = {rq, rk, rv, ra, rb, rsi, rzi};
    for (const Range &r : ins)
        if (ro.overlaps(r)) return GDN_ERR_ALIAS;
    // state_out may share state_in's buffer exactly (in-place update), z_out z_in's
    const Range *outs[] = {&rso, &rzo};
    for (int o = 0; o < 2; ++o) {
        const Range &r = *outs[o];
        if (!r.valid()) continue;
        const int own = o == 0 ? 5 : 6;
        for (int i = 0; i < 7; ++i) {
            if (!r.overlaps(ins[i])) continue;
            if (i != own || r.lo != ins[i].lo) return GDN_ERR_ALIAS;
        }
        if (r.overlaps(ro)) return GDN_ERR_ALIAS;
    }
    if (rso.overlaps(rzo)) return GDN_ERR_ALIAS;
    if (a.fused) {
        if (!a.gate || !a.w_o || !a.gain_q || !a.gain_k || !a.rope_freq || !a.rope_axis) return GDN_ERR_NULL;
        if (a.lat_w < 1) return GDN_ERR_SHAPE;
        if (!a.norm) return GDN_ERR_UNSUPPORTED;
        if (misaligned(a.gate) || misaligned(a.w_o) || misaligned(a.gain_q) || misaligned(a.gain_k) ||
            misaligned(a.rope_freq) || misaligned(a.rope_axis))
            return GDN_ERR_ALIGN;
        const Range extra[] = {range(a.gate, ntok * a.Dv * esz), range(a.w_o, (size_t)a.H * a.Dv * a.Dv * esz),
                               range(a.gain_q, (size_t)a.H * a.Dk * 4), range(a.gain_k, (size_t)a.H * a.Dk * 4),
                               range(a.rope_freq, (size_t)a.Dk / 2 * 4), range(a.rope_axis, (size_t)a.Dk / 2 * 4)};
        for (const Range &r : extra)
            if (ro.overlaps(r) || rso.overlaps(r) || rzo.overlaps(r)) return GDN_ERR_ALIAS;
    }
    return GDN_OK;
}

template <class E>
gdn::FrameParams<E> make_frame_params(const FrameArgs &a, int NS, void *ws) {
    gdn::FrameParams<E> p;
    p.q = (const E *)a.q;
    p.k = (const E *)a.k;
    p.v = (const E *)a.v;
    p.alpha = a.alpha;
    p.beta = a.beta;
    p.state_in = a.state_in;
    p.out = (E *)a.out;
    p.state_out = a.state_out;
    p.B = a.B;
    p.H = a.H;
    p.F = a.F;
    p.N = a.N;
    p.NS = NS;
    p.NBT = 64 * ((frame_blocks(a.N) + NS - 1) / NS);
    frame_out_split((long long)a.B * a.H * a.F, a.N, gdn::kFrameOutWgs, p.OB, p.OTPW);
    p.key_scale = a.key_scale;
    p.z_in = a.norm ? a.z_in : nullptr;
    p.z_out = a.norm ? a.z_out : nullptr;
    p.eps = a.eps;
    const FrameWs L = frame_ws_layout(a.B, a.H, a.F, a.Dk, a.Dv, sizeof(E), NS,
                                      frame_feat_rows(a.fused, a.bf16, a.B, a.H, a.F, a.N));
    unsigned char *base = (unsigned char *)ws;
    p.PG = (float *)(base + L.PG);
    p.PA = (float *)(base + L.PA);
    p.Gf = (E *)(base + L.Gf);
    p.Af = (float *)(base + L.Af);
    p.Hf = (E *)(base + L.Hf);
    p.Hb = (float *)(base + L.Hb);
    p.PGz = (float *)(base + L.PGz);
    p.Gzf = (E *)(base + L.Gzf);
    p.rope = (float *)(base + L.FQ);
    p.fkt = (float *)(base + L.FKT);
    p.fkh = (float *)(base + L.FKH);
    p.no_z = 0;
    p.gate = (const E *)a.gate;
    p.w_o = (const E *)a.w_o;
    p.gain_q = a.gain_q;
    p.gain_k = a.gain_k;
    p.rope_freq = a.rope_freq;
    p.rope_axis = a.rope_axis;
    p.rms_eps = a.rms_eps;
    p.lat_w = a.lat_w;
    p.t0 = a.t0;
    p.feat_scale = a.key_scale;
    if (a.fused) {
        // the key scale is applied to the key features as they are formed
        p.key_scale = 1.f;
        // at most 256 workgroups in all, one per CU, unless the units alone exceed
        // that: each stages H_f and W_o anew (D = 128: 70 KB in bf16, where 480
        // workgroups of 8 waves took 36.0 us against 32.5; 137 KB in fp32, where
        // only one fits a CU; D = 64: 18 and 36 KB, other counts not measured)
        const long long units = (long long)a.B * a.H * a.F;
        const int ntf = (a.N + 15) / 16;
        long long ob = 256 / units;
        if (ob < 1) ob = 1;
        if (ob > ntf) ob = ntf;
        p.OTPW = (int)((ntf + ob - 1) / ob);
        p.OB = (ntf + p.OTPW - 1) / p.OTPW;
    }
    return p;
}

constexpr int kFrameStages = 4;  // summaries, reduction, scan, output

template <class E, int DK, int DV, bool NORM, bool BIDIR, bool FUSED = false>
hipError_t launch_frame(const gdn::FrameParams<E> &p, hipStream_t s, int reps, hipEvent_t *ev) {
    using LS = gdn::FrameSumLds<E, DK, DV, FUSED>;
    using LO = gdn::FrameOutLds<E, DK, DV, NORM>;
    using LF = gdn::FusedOutLds<DK, DV>;
    const void *out_kernel;
    size_t out_lds;
    if constexpr (FUSED) {
        out_kernel = (const void *)gdn::gdn_frame_output_fused_kernel<DK, DV>;
        out_lds = LF::bytes;
    } else {
        out_kernel = (const void *)gdn::gdn_frame_output_kernel<E, DK, DV, NORM>;
        out_lds = LO::bytes;
    }
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] {
        hipError_t e = hipFuncSetAttribute((const void *)gdn::gdn_frame_summary_kernel<E, DK, DV, NORM, FUSED>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)LS::bytes);
        if (e == hipSuccess)
            e = hipFuncSetAttribute(out_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)out_lds);
        attr_err = e;
    });
    if (attr_err != hipSuccess) return attr_err;
    const long long BH = (long long)p.B * p.H, units = BH * p.F;
    constexpr int NJ = DV / 16 + NORM;
    // reduction items per unit (FUSED: also the unrotated-key G fragments)
    constexpr int NI = (DK / 16) * (DK / 32) * (FUSED ? 2 : 1) + (DK / 16) * NJ;
    auto stage = [&](int i) -> hipError_t {
        switch (i) {
        case 0:
            return launch((const void *)gdn::gdn_frame_summary_kernel<E, DK, DV, NORM, FUSED>,
                          dim3((unsigned)(units * p.NS)), dim3(gdn::sum_threads<FUSED>()), LS::bytes, s, p);
        case 1:
            // a single split writes the summaries in their final form
            if (p.NS > 1)
                return launch((const void *)gdn::gdn_frame_reduce_kernel<E, DK, DV, NORM, FUSED>,
                              dim3((unsigned)units, (NI + 3) / 4), dim3(256), 0, s, p);
            return hipSuccess;
        case 2:
            return launch((const void *)gdn::gdn_frame_scan_kernel<E, DK, DV, NORM, BIDIR, FUSED>,
                          dim3(gdn::xcd_blocks(BH, NJ)), dim3(64), 0, s, p);
        default:
            if constexpr (FUSED)
                return launch((const void *)gdn::gdn_frame_output_fused_kernel<DK, DV>,
                              dim3(gdn::xcd_blocks(units, p.OB)), dim3(gdn::kFusedOutWaves * 64), LF::bytes, s, p);
            else
                return launch((const void *)gdn::gdn_frame_output_kernel<E, DK, DV, NORM>,
                              dim3(gdn::xcd_blocks(units, p.OB)), dim3(LO::WAVES * 64), LO::bytes, s, p);
        }
    };
    hipError_t er = hipSuccess;
    for (int i = 0; i < kFrameStages && er == hipSuccess; ++i) {
        if (!ev) {
            er = stage(i);
            continue;
        }
        er = hipEventRecord(ev[2 * i], s);
        for (int r = 0; r < reps && er == hipSuccess; ++r) er = stage(i);
        if (er == hipSuccess) er = hipEventRecord(ev[2 * i + 1], s);
    }
    return er;
}

// The fused operator in fp32: the rotation table and the key features, then the
// summaries on the rotated keys (G, A) and on the unrotated ones (the normalizer's
// Gram matrix and K~^T beta), the fused reduction and scan, and the fp32 output
// (query features, readout, gate, projection).  The four
// profiled stages are: features and summaries, reduction, scan, output and
// projection.
template <int DK, int DV, bool BIDIR>
hipError_t launch_frame_fused32(const gdn::FrameParams<float> &p, hipStream_t s, int reps, hipEvent_t *ev) {
    using E = float;
    using LS = gdn::FrameSumLds<E, DK, DV, false>;
    using LO = gdn::FusedOut32Lds<DK, DV>;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [&] {
        hipError_t e = hipFuncSetAttribute((const void *)gdn::gdn_frame_summary_kernel<E, DK, DV, true, false>,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)LS::bytes);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)gdn::gdn_frame_summary_kernel<E, DK, DV, true, false, true>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)LS::bytes);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)gdn::gdn_frame_output_fused32_kernel<DK, DV>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, (int)LO::bytes);
        attr_err = e;
    });
    if (attr_err != hipSuccess) return attr_err;
    const long long BH = (long long)p.B * p.H, units = BH * p.F;
    constexpr int NJ = DV / 16 + 1;
    constexpr int NI = (DK / 16) * (DK / 32) * 2 + (DK / 16) * NJ;
    const size_t rows = (size_t)BH * p.F * p.N;                     // key rows
    const size_t feat_blocks = (rows * (DK / 4) + 255) / 256;
    const int lat_rows = 1 + (p.N - 1) / p.lat_w, lat_cols = p.N < p.lat_w ? p.N : p.lat_w;
    int rope_rows = p.F + (lat_rows > lat_cols ? lat_rows : lat_cols);
    auto stage = [&](int i) -> hipError_t {
        switch (i) {
        case 0: {
            gdn::FrameParams<E> copy = p;
            void *args[] = {&copy, &rope_rows};
            hipError_t e = hipLaunchKernel((const void *)gdn::gdn_frame_rope_kernel<DK>,
                                           dim3((unsigned)(((long long)rope_rows * (DK / 2) + 255) / 256)), dim3(256), args,
                                           0, s);
            if (e == hipSuccess)
                e = launch((const void *)gdn::gdn_frame_kfeatures_kernel<DK>, dim3((unsigned)feat_blocks), dim3(256), 0, s,
                           p);
            // rotated keys: G and the A tiles
            gdn::FrameParams<E> pr = p;
            pr.k = p.fkh;
            pr.no_z = 1;
            if (e == hipSuccess)
                e = launch((const void *)gdn::gdn_frame_summary_kernel<E, DK, DV, true, false>,
                           dim3((unsigned)(units * p.NS)), dim3(gdn::sum_threads<false>()), LS::bytes, s, pr);
            // unrotated keys: their Gram matrix, the normalizer tile
            gdn::FrameParams<E> pu = p;
            pu.k = p.fkt;
            if (e == hipSuccess)
                e = launch((const void *)gdn::gdn_frame_summary_kernel<E, DK, DV, true, false, true>,
                           dim3((unsigned)(units * p.NS)), dim3(gdn::sum_threads<false>()), LS::bytes, s, pu);
            return e;
        }
        case 1:
            if (p.NS > 1)
                return launch((const void *)gdn::gdn_frame_reduce_kernel<E, DK, DV, true, true>,
                              dim3((unsigned)units, (NI + 3) / 4), dim3(256), 0, s, p);
            return hipSuccess;
        case 2:
            return launch((const void *)gdn::gdn_frame_scan_kernel<E, DK, DV, true, BIDIR, true>,
                          dim3(gdn::xcd_blocks(BH, NJ)), dim3(64), 0, s, p);
        default:
            return launch((const void *)gdn::gdn_frame_output_fused32_kernel<DK, DV>, dim3(gdn::xcd_blocks(units, p.OB)),
                          dim3(gdn::kFusedOutWaves32 * 64), LO::bytes, s, p);
        }
    };
    hipError_t er = hipSuccess;
    for (int i = 0; i < kFrameStages && er == hipSuccess; ++i) {
        if (!ev) {
            er = stage(i);
            continue;
        }
        er = hipEventRecord(ev[2 * i], s);
        for (int r = 0; r < reps && er == hipSuccess; ++r) er = stage(i);
        if (er == hipSuccess) er = hipEventRecord(ev[2 * i + 1], s);
    }
    return er;
}

template <bool BIDIR>
hipError_t frame_dispatch_fused32(const gdn::FrameParams<float> &p, int Dk, int Dv, hipStream_t s, int reps,
                                  hipEvent_t *ev) {
    if (Dk == 128 && Dv == 128) return launch_frame_fused32<128, 128, BIDIR>(p, s, reps, ev);
    if (Dk == 64 && Dv == 64) return launch_frame_fused32<64, 64, BIDIR>(p, s, reps, ev);
    if (Dk == 128 && Dv == 64) return launch_frame_fused32<128, 64, BIDIR>(p, s, reps, ev);
    return launch_frame_fused32<64, 128, BIDIR>(p, s, reps, ev);
}

template <class E, bool NORM, bool BIDIR, bool FUSED = false>
hipError_t frame_dispatch_n(const gdn::FrameParams<E> &p, int Dk, int Dv, hipStream_t s, int reps, hipEvent_t *ev) {
    if (Dk == 128 && Dv == 128) return launch_frame<E, 128, 128, NORM, BIDIR, FUSED>(p, s, reps, ev);
    if (Dk == 64 && Dv == 64) return launch_frame<E, 64, 64, NORM, BIDIR, FUSED>(p, s, reps, ev);
    if (Dk == 128 && Dv == 64) return launch_frame<E, 128, 64, NORM, BIDIR, FUSED>(p, s, reps, ev);
    return launch_frame<E, 64, 128, NORM, BIDIR, FUSED>(p, s, reps, ev);
}

template <class E>
hipError_t frame_dispatch(const FrameArgs &a, int NS, void *ws, hipStream_t s, int reps, hipEvent_t *ev) {
    const gdn::FrameParams<E> p = make_frame_params<E>(a, NS, ws);
    if constexpr (sizeof(E) == 2) {
        if (a.fused)
            return a.bidir ? frame_dispatch_n<E, true, true, true>(p, a.Dk, a.Dv, s, reps, ev)
                           : frame_dispatch_n<E, true, false, true>(p, a.Dk, a.Dv, s, reps, ev);
    } else {
        if (a.fused)
            return a.bidir ? frame_dispatch_fused32<true>(p, a.Dk, a.Dv, s, reps, ev)
                           : frame_dispatch_fused32<false>(p, a.Dk, a.Dv, s, reps, ev);
    }
    if (a.bidir)
        return a.norm ? frame_dispatch_n<E, true, true>(p, a.Dk, a.Dv, s, reps, ev)
                      : frame_dispatch_n<E, false, true>(p, a.Dk, a.Dv, s, reps, ev);
    return a.norm ? frame_dispatch_n<E, true, false>(p, a.Dk, a.Dv, s, reps, ev)
                  : frame_dispatch_n<E, false, false>(p, a.Dk, a.Dv, s, reps, ev);
}

int frame_run(const FrameArgs &a, int token_splits, void *ws, size_t ws_bytes, void *stream, int reps,
              hipEvent_t *ev) {
    int st = frame_validate(a);
    if (st != GDN_OK) return st;
    const int NS = frame_splits((long long)a.B * a.H * a.F, a.N, token_splits);
    if (!ws || ((uintptr_t)ws & 255u) ||
        ws_bytes < frame_ws_layout(a.B, a.H, a.F, a.Dk, a.Dv, a.bf16 ? 2 : 4, NS,
                                   frame_feat_rows(a.fused, a.bf16, a.B, a.H, a.F, a.N))
                       .total)
        return GDN_ERR_WORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    const hipError_t e = a.bf16 ? frame_dispatch<uint16_t>(a, NS, ws, s, reps, ev)
                                : frame_dispatch<float>(a, NS, ws, s, reps, ev);
    return e == hipSuccess ? GDN_OK : GDN_ERR_HIP;
}

int frame_run_cached(const FrameArgs &a, void *stream) {
    int st = frame_validate(a);
    if (st != GDN_OK) return st;
    const size_t need = frame_ws_layout(a.B, a.H, a.F, a.Dk, a.Dv, a.bf16 ? 2 : 4,
                                        frame_splits((long long)a.B * a.H * a.F, a.N, 0),
                                        frame_feat_rows(a.fused, a.bf16, a.B, a.H, a.F, a.N))
                            .total;
    void *ws = nullptr;
    st = cached_workspace(need, &ws);
    if (st != GDN_OK) return st;
    return frame_run(a, 0, ws, need, stream, 1, nullptr);
}

int frame_profile(const FrameArgs &a, int token_splits, void *ws, size_t ws_bytes, int reps, float *stage_ms,
                  void *stream) {
    if (!stage_ms || reps < 1) return GDN_ERR_NULL;
    // stages are re-run in place, so no state may be updated in place
    if (a.state_in && a.state_in == a.state_out) return GDN_ERR_ALIAS;
    if (a.norm && a.z_in && a.z_in == a.z_out) return GDN_ERR_ALIAS;
    hipEvent_t ev[2 * kFrameStages] = {};
    int status = GDN_OK;
    for (auto &e : ev)
        if (status == GDN_OK && hipEventCreate(&e) != hipSuccess) {
            e = nullptr;
            status = GDN_ERR_HIP;
        }
    if (status == GDN_OK) status = frame_run(a, token_splits, ws, ws_bytes, stream, reps, ev);
    if (status == GDN_OK && hipStreamSynchronize((hipStream_t)stream) != hipSuccess) status = GDN_ERR_HIP;
    for (int i = 0; i < kFrameStages && status == GDN_OK; ++i) {
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, ev[2 * i], ev[2 * i + 1]) != hipSuccess) status = GDN_ERR_HIP;
        stage_ms[i] = ms / reps;
    }
    for (auto &e : ev)
        if (e) (void)hipEventDestroy(e);
    return status;
}

FrameArgs frame_args(const void *q, const void *k, const void *v, const float *alpha, const float *beta,
                     const float *state_in, const float *z_in, void *out, float *state_out, float *z_out, int B,
                     int H, int F, int N, int Dk, int Dv, float key_scale, float eps, bool bf16, bool norm,
                     bool bidir = false) {
    return FrameArgs{q, k, v, alpha, beta, state_in, z_in, out, state_out, z_out,
                     B, H, F, N, Dk, Dv, key_scale, eps, bf16, norm, bidir};
}

FrameArgs fused_args(const void *q_raw, const void *k_raw, const void *v, const void *gate, const void *w_o,
                     const float *alpha, const float *beta, const float *gain_q, const float *gain_k,
                     const float *rope_freq, const int *rope_axis, const float *state_in, const float *z_in,
                     void *out, float *state_out, float *z_out, int B, int H, int F, int N, int Dk, int Dv,
                     int lat_w, int t0, float key_scale, float rms_eps, float eps, int bidirectional,
                     bool bf16 = true) {
    FrameArgs a = frame_args(q_raw, k_raw, v, alpha, beta, state_in, z_in, out, state_out, z_out, B, H, F, N, Dk,
                             Dv, key_scale, eps, bf16, true, bidirectional != 0);
    a.fused = true;
    a.gate = gate;
    a.w_o = w_o;
    a.gain_q = gain_q;
    a.gain_k = gain_k;
    a.rope_freq = rope_freq;
    a.rope_axis = rope_axis;
    a.rms_eps = rms_eps;
    a.lat_w = lat_w;
    a.t0 = t0;
    return a;
}

}  // namespace

extern "C" {

int gdn_chunk_forward(const void *q, const void *k, const void *v, const float *alpha,
                      const float *beta, const float *state_in, void *out, float *state_out, int B,
                      int H, int T, int Dk, int Dv, int chunk, void *stream) {
    return run_cached(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk, true,
                      stream);
}

int gdn_chunk_forward_f32(const float *q, const float *k, const float *v, const float *alpha,
                          const float *beta, const float *state_in, float *out, float *state_out,
                          int B, int H, int T, int Dk, int Dv, int chunk, void *stream) {
    return run_cached(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk, false,
                      stream);
}

int gdn_workspace_check(int B, int H, int T, int Dk, int Dv, int chunk, int is_bf16, int scan_group) {
    if (!shape_ok(B, H, T)) return GDN_ERR_SHAPE;
    if (!dims_ok(Dk, Dv, chunk)) return GDN_ERR_UNSUPPORTED;
    const size_t esz = is_bf16 ? 2 : 4;
    const int G = resolve_group(num_chunks(T), (long long)B * H, Dv, scan_group, is_bf16 != 0);
    const WsLayout L = ws_layout(B, H, T, Dk, Dv, esz, G);
    const WsNeeds n = ws_needs(B, H, T, Dk, Dv, esz, G);
    const size_t start[] = {L.er, L.gf, L.W, L.Ut, L.Hs, L.Us, L.Nf, L.PsiT, L.lgam, L.HgT, L.total};
    const size_t need[] = {n.er, n.gf, n.W, n.Ut, n.Hs, n.Us, n.Nf, n.PsiT, n.lgam, n.HgT};
    for (int r = 0; r < 10; ++r) {
        if (start[r] % 256) return r + 1;                    // regions start 256-byte aligned
        if (need[r] > start[r + 1] - start[r]) return r + 1;  // region too small
    }
    return GDN_OK;
}

int gdn_chunk_forward_noalloc(const void *q, const void *k, const void *v, const float *alpha,
                              const float *beta, const float *state_in, void *out, float *state_out, int B,
                              int H, int T, int Dk, int Dv, int chunk, void *stream) {
    return run_noalloc(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk, stream);
}

size_t gdn_workspace_bytes(int B, int H, int T, int Dk, int Dv, int chunk, int is_bf16) {
    return gdn_workspace_bytes_ex(B, H, T, Dk, Dv, chunk, is_bf16, 0);
}

int gdn_scan_group_size(int B, int H, int T, int Dk, int Dv, int chunk, int is_bf16, int scan_group) {
    if (!shape_ok(B, H, T) || !dims_ok(Dk, Dv, chunk)) return 0;
    return resolve_group(num_chunks(T), (long long)B * H, Dv, scan_group, is_bf16 != 0);
}

size_t gdn_workspace_bytes_ex(int B, int H, int T, int Dk, int Dv, int chunk, int is_bf16,
                              int scan_group) {
    if (!shape_ok(B, H, T) || !dims_ok(Dk, Dv, chunk)) return 0;
    return ws_layout(B, H, T, Dk, Dv, is_bf16 ? 2 : 4,
                     resolve_group(num_chunks(T), (long long)B * H, Dv, scan_group, is_bf16 != 0))
        .total;
}

int gdn_chunk_forward_ws(const void *q, const void *k, const void *v, const float *alpha,
                         const float *beta, const float *state_in, void *out, float *state_out,
                         int B, int H, int T, int Dk, int Dv, int chunk, void *ws, size_t ws_bytes,
                         void *stream) {
    return run(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk, true, 0, ws,
               ws_bytes, stream, nullptr);
}

int gdn_chunk_forward_f32_ws(const float *q, const float *k, const float *v, const float *alpha,
                             const float *beta, const float *state_in, float *out, float *state_out,
                             int B, int H, int T, int Dk, int Dv, int chunk, void *ws,
                             size_t ws_bytes, void *stream) {
    return run(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk, false, 0, ws,
               ws_bytes, stream, nullptr);
}

int gdn_chunk_forward_ex(const void *q, const void *k, const void *v, const float *alpha,
                         const float *beta, const float *state_in, void *out, float *state_out,
                         int B, int H, int T, int Dk, int Dv, int chunk, int is_bf16, int scan_group,
                         void *ws, size_t ws_bytes, void *stream) {
    return run(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk, is_bf16 != 0,
               scan_group, ws, ws_bytes, stream, nullptr);
}

int gdn_profile_stages(const void *q, const void *k, const void *v, const float *alpha,
                       const float *beta, const float *state_in, void *out, float *state_out,
                       int B, int H, int T, int Dk, int Dv, int chunk, int is_bf16, int scan_group,
                       void *ws, size_t ws_bytes, int reps, float *stage_ms, void *stream) {
    if (!stage_ms || reps < 1) return GDN_ERR_NULL;
    // Stages are re-run in place, so the state may not be updated in place.
    if (state_in && state_in == state_out) return GDN_ERR_ALIAS;
    StageTiming tm{};
    tm.reps = reps;
    int status = GDN_OK;
    for (auto &e : tm.ev)
        if (status == GDN_OK && hipEventCreate(&e) != hipSuccess) {
            e = nullptr;
            status = GDN_ERR_HIP;
        }
    if (status == GDN_OK)
        status = run(q, k, v, alpha, beta, state_in, out, state_out, B, H, T, Dk, Dv, chunk,
                     is_bf16 != 0, scan_group, ws, ws_bytes, stream, &tm);
    if (status == GDN_OK && hipStreamSynchronize((hipStream_t)stream) != hipSuccess)
        status = GDN_ERR_HIP;
    if (status == GDN_OK) {
        for (int i = 0; i < kStages; ++i) stage_ms[i] = tm.ms[i];
        stage_ms[kStages] = 0.f;                 // once the output's, which stage 3 now forms
    }
    for (auto &e : tm.ev)
        if (e) (void)hipEventDestroy(e);
    return status;
}

int gdn_frame_forward(const void *q, const void *k, const void *v, const float *alpha, const float *beta,
                      const float *state_in, void *out, float *state_out, int B, int H, int F, int N,
                      int Dk, int Dv, float key_scale, void *stream) {
    return frame_run_cached(frame_args(q, k, v, alpha, beta, state_in, nullptr, out, state_out, nullptr, B, H,
                                       F, N, Dk, Dv, key_scale, 0.f, true, false),
                            stream);
}

int gdn_frame_forward_f32(const float *q, const float *k, const float *v, const float *alpha,
                          const float *beta, const float *state_in, float *out, float *state_out, int B,
                          int H, int F, int N, int Dk, int Dv, float key_scale, void *stream) {
    return frame_run_cached(frame_args(q, k, v, alpha, beta, state_in, nullptr, out, state_out, nullptr, B, H,
                                       F, N, Dk, Dv, key_scale, 0.f, false, false),
                            stream);
}

int gdn_frame_token_splits(int B, int H, int F, int N, int Dk, int Dv, int token_splits) {
    if (!frame_shape_ok(B, H, F, N) || !frame_dims_ok(Dk, Dv)) return 0;
    return frame_splits((long long)B * H * F, N, token_splits);
}

size_t gdn_frame_workspace_bytes(int B, int H, int F, int N, int Dk, int Dv, int is_bf16, int token_splits) {
    if (!frame_shape_ok(B, H, F, N) || !frame_dims_ok(Dk, Dv)) return 0;
    return frame_ws_layout(B, H, F, Dk, Dv, is_bf16 ? 2 : 4, frame_splits((long long)B * H * F, N, token_splits))
        .total;
}

int gdn_frame_forward_ex(const void *q, const void *k, const void *v, const float *alpha, const float *beta,
                         const float *state_in, void *out, float *state_out, int B, int H, int F, int N,
                         int Dk, int Dv, float key_scale, int is_bf16, int token_splits, void *ws,
                         size_t ws_bytes, void *stream) {
    return frame_run(frame_args(q, k, v, alpha, beta, state_in, nullptr, out, state_out, nullptr, B, H, F, N,
                                Dk, Dv, key_scale, 0.f, is_bf16 != 0, false),
                     token_splits, ws, ws_bytes, stream, 1, nullptr);
}

int gdn_frame_profile_stages(const void *q, const void *k, const void *v, const float *alpha,
                             const float *beta, const float *state_in, void *out, float *state_out, int B,
                             int H, int F, int N, int Dk, int Dv, float key_scale, int is_bf16,
                             int token_splits, void *ws, size_t ws_bytes, int reps, float *stage_ms,
                             void *stream) {
    return frame_profile(frame_args(q, k, v, alpha, beta, state_in, nullptr, out, state_out, nullptr, B, H, F,
                                    N, Dk, Dv, key_scale, 0.f, is_bf16 != 0, false),
                         token_splits, ws, ws_bytes, reps, stage_ms, stream);
}

int gdn_frame_forward_norm(const void *q, const void *k, const void *v, const float *alpha, const float *beta,
                           const float *state_in, const float *z_in, void *out, float *state_out, float *z_out,
                           int B, int H, int F, int N, int Dk, int Dv, float key_scale, float eps, int is_bf16,
                           void *stream) {
    return frame_run_cached(frame_args(q, k, v, alpha, beta, state_in, z_in, out, state_out, z_out, B, H, F, N,
                                       Dk, Dv, key_scale, eps, is_bf16 != 0, true),
                            stream);
}

int gdn_frame_forward_norm_ex(const void *q, const void *k, const void *v, const float *alpha,
                              const float *beta, const float *state_in, const float *z_in, void *out,
                              float *state_out, float *z_out, int B, int H, int F, int N, int Dk, int Dv,
                              float key_scale, float eps, int is_bf16, int token_splits, void *ws,
                              size_t ws_bytes, void *stream) {
    return frame_run(frame_args(q, k, v, alpha, beta, state_in, z_in, out, state_out, z_out, B, H, F, N, Dk, Dv,
                                key_scale, eps, is_bf16 != 0, true),
                     token_splits, ws, ws_bytes, stream, 1, nullptr);
}

int gdn_frame_profile_stages_norm(const void *q, const void *k, const void *v, const float *alpha,
                                  const float *beta, const float *state_in, const float *z_in, void *out,
                                  float *state_out, float *z_out, int B, int H, int F, int N, int Dk, int Dv,
                                  float key_scale, float eps, int is_bf16, int token_splits, void *ws,
                                  size_t ws_bytes, int reps, float *stage_ms, void *stream) {
    return frame_profile(frame_args(q, k, v, alpha, beta, state_in, z_in, out, state_out, z_out, B, H, F, N, Dk,
                                    Dv, key_scale, eps, is_bf16 != 0, true),
                         token_splits, ws, ws_bytes, reps, stage_ms, stream);
}

int gdn_frame_forward_bidir(const void *q, const void *k, const void *v, const float *alpha, const float *beta,
                            const float *state_in, const float *z_in, void *out, float *state_out,
                            float *z_out, int B, int H, int F, int N, int Dk, int Dv, float key_scale, float eps,
                            int is_bf16, int normalized, void *stream) {
    return frame_run_cached(frame_args(q, k, v, alpha, beta, state_in, z_in, out, state_out, z_out, B, H, F, N,
                                       Dk, Dv, key_scale, eps, is_bf16 != 0, normalized != 0, true),
                            stream);
}

int gdn_frame_forward_bidir_ex(const void *q, const void *k, const void *v, const float *alpha,
                               const float *beta, const float *state_in, const float *z_in, void *out,
                               float *state_out, float *z_out, int B, int H, int F, int N, int Dk, int Dv,
                               float key_scale, float eps, int is_bf16, int normalized, int token_splits,
                               void *ws, size_t ws_bytes, void *stream) {
    return frame_run(frame_args(q, k, v, alpha, beta, state_in, z_in, out, state_out, z_out, B, H, F, N, Dk, Dv,
                                key_scale, eps, is_bf16 != 0, normalized != 0, true),
                     token_splits, ws, ws_bytes, stream, 1, nullptr);
}

int gdn_frame_profile_stages_bidir(const void *q, const void *k, const void *v, const float *alpha,
                                   const float *beta, const float *state_in, const float *z_in, void *out,
                                   float *state_out, float *z_out, int B, int H, int F, int N, int Dk, int Dv,
                                   float key_scale, float eps, int is_bf16, int normalized, int token_splits,
                                   void *ws, size_t ws_bytes, int reps, float *stage_ms, void *stream) {
    return frame_profile(frame_args(q, k, v, alpha, beta, state_in, z_in, out, state_out, z_out, B, H, F, N, Dk,
                                    Dv, key_scale, eps, is_bf16 != 0, normalized != 0, true),
                         token_splits, ws, ws_bytes, reps, stage_ms, stream);
}

int gdn_frame_forward_fused(const void *q_raw, const void *k_raw, const void *v, const void *gate,
                            const void *w_o, const float *alpha, const float *beta, const float *gain_q,
                            const float *gain_k, const float *rope_freq, const int *rope_axis,
                            const float *state_in, const float *z_in, void *out, float *state_out, float *z_out,
                            int B, int H, int F, int N, int Dk, int Dv, int lat_w, int t0, float key_scale,
                            float rms_eps, float eps, int bidirectional, void *stream) {
    return frame_run_cached(fused_args(q_raw, k_raw, v, gate, w_o, alpha, beta, gain_q, gain_k, rope_freq,
                                       rope_axis, state_in, z_in, out, state_out, z_out, B, H, F, N, Dk, Dv, lat_w,
                                       t0, key_scale, rms_eps, eps, bidirectional),
                            stream);
}

int gdn_frame_forward_fused_ex(const void *q_raw, const void *k_raw, const void *v, const void *gate,
                               const void *w_o, const float *alpha, const float *beta, const float *gain_q,
                               const float *gain_k, const float *rope_freq, const int *rope_axis,
                               const float *state_in, const float *z_in, void *out, float *state_out,
                               float *z_out, int B, int H, int F, int N, int Dk, int Dv, int lat_w, int t0,
                               float key_scale, float rms_eps, float eps, int bidirectional, int token_splits,
                               void *ws, size_t ws_bytes, void *stream) {
    return frame_run(fused_args(q_raw, k_raw, v, gate, w_o, alpha, beta, gain_q, gain_k, rope_freq, rope_axis,
                                state_in, z_in, out, state_out, z_out, B, H, F, N, Dk, Dv, lat_w, t0, key_scale,
                                rms_eps, eps, bidirectional),
                     token_splits, ws, ws_bytes, stream, 1, nullptr);
}

int gdn_frame_profile_stages_fused(const void *q_raw, const void *k_raw, const void *v, const void *gate,
                                   const void *w_o, const float *alpha, const float *beta, const float *gain_q,
                                   const float *gain_k, const float *rope_freq, const int *rope_axis,
                                   const float *state_in, const float *z_in, void *out, float *state_out,
                                   float *z_out, int B, int H, int F, int N, int Dk, int Dv, int lat_w, int t0,
                                   float key_scale, float rms_eps, float eps, int bidirectional,
                                   int token_splits, void *ws, size_t ws_bytes, int reps, float *stage_ms,
                                   void *stream) {
    return frame_profile(fused_args(q_raw, k_raw, v, gate, w_o, alpha, beta, gain_q, gain_k, rope_freq,
                                    rope_axis, state_in, z_in, out, state_out, z_out, B, H, F, N, Dk, Dv, lat_w, t0,
                                    key_scale, rms_eps, eps, bidirectional),
                         token_splits, ws, ws_bytes, reps, stage_ms, stream);
}

int gdn_frame_forward_fused_f32(const float *q_raw, const float *k_raw, const float *v, const float *gate,
                                const float *w_o, const float *alpha, const float *beta, const float *gain_q,
                                const float *gain_k, const float *rope_freq, const int *rope_axis,
                                const float *state_in, const float *z_in, float *out, float *state_out,
                                float *z_out, int B, int H, int F, int N, int Dk, int Dv, int lat_w, int t0,
                                float key_scale, float rms_eps, float eps, int bidirectional, void *stream) {
    return frame_run_cached(fused_args(q_raw, k_raw, v, gate, w_o, alpha, beta, gain_q, gain_k, rope_freq,
                                       rope_axis, state_in, z_in, out, state_out, z_out, B, H, F, N, Dk, Dv, lat_w,
                                       t0, key_scale, rms_eps, eps, bidirectional, false),
                            stream);
}

int gdn_frame_forward_fused_f32_ex(const float *q_raw, const float *k_raw, const float *v, const float *gate,
                                   const float *w_o, const float *alpha, const float *beta, const float *gain_q,
                                   const float *gain_k, const float *rope_freq, const int *rope_axis,
                                   const float *state_in, const float *z_in, float *out, float *state_out,
                                   float *z_out, int B, int H, int F, int N, int Dk, int Dv, int lat_w, int t0,
                                   float key_scale, float rms_eps, float eps, int bidirectional, int token_splits,
                                   void *ws, size_t ws_bytes, void *stream) {
    return frame_run(fused_args(q_raw, k_raw, v, gate, w_o, alpha, beta, gain_q, gain_k, rope_freq, rope_axis,
                                state_in, z_in, out, state_out, z_out, B, H, F, N, Dk, Dv, lat_w, t0, key_scale,
                                rms_eps, eps, bidirectional, false),
                     token_splits, ws, ws_bytes, stream, 1, nullptr);
}

int gdn_frame_profile_stages_fused_f32(const float *q_raw, const float *k_raw, const float *v, const float *gate,
                                       const float *w_o, const float *alpha, const float *beta,
                                       const float *gain_q, const float *gain_k, const float *rope_freq,
                                       const int *rope_axis, const float *state_in, const float *z_in, float *out,
                                       float *state_out, float *z_out, int B, int H, int F, int N, int Dk, int Dv,
                                       int lat_w, int t0, float key_scale, float rms_eps, float eps,
                                       int bidirectional, int token_splits, void *ws, size_t ws_bytes, int reps,
                                       float *stage_ms, void *stream) {
    return frame_profile(fused_args(q_raw, k_raw, v, gate, w_o, alpha, beta, gain_q, gain_k, rope_freq,
                                    rope_axis, state_in, z_in, out, state_out, z_out, B, H, F, N, Dk, Dv, lat_w, t0,
                                    key_scale, rms_eps, eps, bidirectional, false),
                         token_splits, ws, ws_bytes, reps, stage_ms, stream);
}

size_t gdn_frame_fused_workspace_bytes(int B, int H, int F, int N, int Dk, int Dv, int is_bf16, int token_splits) {
    if (!frame_shape_ok(B, H, F, N) || !frame_dims_ok(Dk, Dv)) return 0;
    return frame_ws_layout(B, H, F, Dk, Dv, is_bf16 ? 2 : 4, frame_splits((long long)B * H * F, N, token_splits),
                           frame_feat_rows(true, is_bf16 != 0, B, H, F, N))
        .total;
}

const char *gdn_status_string(int status) {
    switch (status) {
    case GDN_OK: return "ok";
    case GDN_ERR_NULL: return "a required pointer is NULL";
    case GDN_ERR_SHAPE: return "invalid shape (sizes must be >= 1, B*H <= 65535, token and grid indices within int range)";
    case GDN_ERR_UNSUPPORTED: return "unsupported configuration (Dk, Dv in {64,128}; chunk == 64)";
    case GDN_ERR_WORKSPACE: return "workspace missing, too small or not 256-byte aligned";
    case GDN_ERR_HIP: return "HIP runtime error or kernel launch failure";
    case GDN_ERR_ALIGN: return "a pointer is not 16-byte aligned";
    case GDN_ERR_ALIAS: return "an output overlaps an input";
    default: return "unknown status";
    }
}

}  // extern "C"

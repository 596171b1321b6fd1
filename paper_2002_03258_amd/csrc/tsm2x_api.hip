// C ABI of the tall-and-skinny product library (declared in include/tsm2x.h):
// argument checking (host only, before any HIP call), launch planning,
// workspace management and dispatch to the gfx950 kernels.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstdlib>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <tuple>
#include <string>
#include <vector>

#include "../../include/tsm2x.h"
#include "tsm2x_internal.h"

using namespace tsm;

namespace {

thread_local std::string g_last_hip;

int hip_fail(hipError_t e, const char* what) {
    g_last_hip = std::string(what) + ": " + hipGetErrorString(e);
    return TSM_ERR_HIP;
}

int check_launch(const char* what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, what);
    return TSM_SUCCESS;
}

// A workspace buffer of the library.  Every stream has its own, so that calls
// on different streams stay independent.
struct WsBuf {
    std::mutex mu;           // held until a call has enqueued its last launch
    void* p = nullptr;
    size_t bytes = 0;
    bool captured = false;   // a graph may hold p
    bool dead = false;       // taken out of the table
    uint64_t used = 0;
};
// (stream, tag of the calling thread for the one handle that names a stream
// per thread)
typedef std::pair<hipStream_t, const void*> WsKey;
constexpr size_t kMaxWsBufs = 64;

struct DevState {
    std::map<WsKey, std::shared_ptr<WsBuf>> bufs;
    std::vector<void*> retired;      // outgrown, but held by captured graphs
    uint64_t clock = 0;
    int cus = 0;
};
std::mutex g_mu;             // may be taken with a WsBuf's mutex held; the other way round only tried
std::vector<DevState> g_dev;

DevState* dev_state(int* dev_out) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return nullptr;
    if (dev_out) *dev_out = dev;
    if ((int)g_dev.size() <= dev) g_dev.resize(dev + 1);
    return &g_dev[dev];
}

int cu_count() {
    std::lock_guard<std::mutex> lk(g_mu);
    DevState* d = dev_state(nullptr);
    if (!d) return 256;
    if (d->cus == 0) {
        int v = 0;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, 0) != hipSuccess || v <= 0)
            v = 256;
        int dev = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            v = 256;
        d->cus = v > 0 ? v : 256;
    }
    return d->cus;
}

int64_t env_int(const char* name, int64_t dflt) {
    const char* s = std::getenv(name);
    if (!s || !*s) return dflt;
    return std::strtoll(s, nullptr, 10);
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

bool valid_dtype(int dt) { return dt >= TSM_F64 && dt <= TSM_F16_SPLIT; }
bool plain_dtype(int dt) { return dt == TSM_F64 || dt == TSM_F32; }
int esize(int dt) { return dt == TSM_F64 ? 8 : 4; }

// What picks a kernel's instance: plain types, every column on a 128-byte
// line, or on 64 bytes for a tall matrix of few columns (2^18 rows, 256
// columns, n <= 16; FP64 beyond 128 columns n <= 8: 541440 x 256, n = 16 233 us
// without and 242 with); 16-bit planes, every column on 16 bytes.
bool aligned(const void* p, int64_t ld, int dtype, int64_t m, int64_t k, int64_t n) {
    if (!plain_dtype(dtype)) return ((uintptr_t)p & 15u) == 0 && ld % 8 == 0;
    const bool few = m >= (int64_t)1 << 18 && k <= 256 && n <= (dtype == TSM_F64 && k > 128 ? 8 : 16);
    return line_aligned(p, ld * esize(dtype), few ? 64 : 128);
}

int pow2_ge(int64_t n) {
    int p = 1;
    while (p < n) p <<= 1;
    return p;
}

// ------------------------------------------------------------- plans
// TSM2R plans pinned by the caller, per (m, k, n, dtype); shared by all devices
typedef std::tuple<int64_t, int64_t, int64_t, int> PinKey;
std::mutex g_pin_mu;
std::map<PinKey, NNPin> g_pins;

NNPin pin_of(int64_t m, int64_t k, int64_t n, int dtype) {
    std::lock_guard<std::mutex> lk(g_pin_mu);
    auto it = g_pins.find(PinKey(m, k, n, dtype));
    return it == g_pins.end() ? NNPin{0, -1} : it->second;
}

int plan_nn(int64_t m, int64_t k, int64_t n, int dtype, int cus, bool line, NNPlan* P,
            bool fine = true) {
    const NNPin pin = pin_of(m, k, n, dtype);
    return plan_tsm2r(m, k, n, dtype, cus, line, P, &pin, fine);
}

struct RTPlan {
    int kp;
    int64_t cpb;
    int64_t bx, by;
};

// rowtile: a wavefront owns 16*RL*RG rows; one pass covers up to 32 output
// columns.  For nout <= 32 a persistent grid of about 8 workgroups per CU
// walks the row tiles; wider outputs are also split into column ranges.
RTPlan plan_rowtile(int64_t m, int64_t kin, int64_t nout, int dt, int cus) {
    RTPlan P{};
    const int es = esize(dt);
    const int RL = 16 / es;
    P.kp = kin <= 8 ? 8 : (kin <= 16 ? 16 : 32);
    // row groups per lane of the instance rowtile_dispatch launches
    const int RG = P.kp == 8 ? 2 : (P.kp == 16 && nout > 16 ? 2 : 1);
    const int64_t TR = 16 * RL * RG;
    const int64_t ntiles = cdiv(m, TR);
    const int64_t wblocks = cdiv(ntiles, 4);
    // nout <= 32 (TSM2L): the persistent grid is capped by occupancy at launch.
    // Wide outputs (dA of TSM2R, write-bound): one workgroup per CU, each
    // wavefront keeping one row tile for a long column range.  Measured: the
    // fewer column ranges are written at once, the closer together in time
    // each column's row tiles are written (256 workgroups: FP32 6.0 TB/s;
    // 1024: 4.9 TB/s)
    const int64_t cap = env_int("TSM2X_RT_BLOCKS", (int64_t)cus * (nout > 32 ? 1 : 4));
    if (nout <= 32) {
        P.cpb = nout;
        P.by = 1;
    } else {
        // as many column ranges, each a multiple of 32, as fit the cap with
        // every wavefront on the same number of row tiles (a range more, and
        // some took two: FP32 dA 20096 x 20011, n = 8: 441 us,
        // 309 so; 20011 x 20011: 973 and 470)
        int64_t by = cap / wblocks;
        if (by < 1) by = 1;
        int64_t cpb = cdiv(nout, by);
        cpb = cdiv(cpb, 32) * 32;
        if (cpb < 32) cpb = 32;
        P.cpb = cpb;
        P.by = cdiv(nout, cpb);
    }
    int64_t bx = wblocks;
    int64_t lim = cap / P.by;
    if (lim < 1) lim = 1;
    if (bx > lim) bx = nout > 32 ? cdiv(wblocks, cdiv(wblocks, lim)) : lim;
    if (bx < 1) bx = 1;
    P.bx = bx;
    return P;
}

struct TNPlan {
    int64_t groups;         // 16-column output tiles (a multiple of ct)
    int S;
    int64_t rslice;
    int ct;                 // output tiles per workgroup
    int pf;                 // 16-bit forms: the next step's X held in flight
    bool yt;                // bf16 planes, n > 16: Y split once into packed terms
    size_t yt_off;          // their offset in the workspace
    size_t ws;
};

// Time of a grid of W equal workgroups relative to the same work spread evenly
// over the `cus` compute units.  A CU takes hardly more than its share of the
// memory bandwidth, however many workgroups it holds, so the grid lasts as
// long as the CUs with one workgroup more than the others; with at most one
// workgroup per CU nothing overlaps the ends of its loop (5 %).
double grid_time(int64_t W, int cus) {
    return W <= cus ? 1.05 * cus / (double)W : (double)(cdiv(W, cus) * cus) / (double)W;
}

// Plain types: one workgroup per ct 16-column tiles (of the output rows) and
// slice of R; its 4 wavefronts split the slice, each with its next step in
// flight.  n > 16: two tiles, which share each staged Y, and one stage of rows
// per step; n <= 16: two tiles and one stage, or one tile and two stages,
// whichever grid takes less time (two tiles read 3-7 % faster; FP32 4096^2,
// n = 8, 128 or 256 workgroups: 17.5 and 14.2 us).  The split S takes the least time
// by grid_time, the two steps a wavefront spends on filling its pipeline and
// on the sums, and the partials; at least two steps per wavefront.  (Before:
// two tiles, S for two workgroups per CU and at least eight steps, nothing in
// flight for n <= 16.  FP32 20032^2, n = 8: 358 us, now 247; 4096^2: 24 and
// 14; 3001^2: 43 and 13; FP64 20011^2, n = 16: 868 and 643.)
void plan_tn_plain(int64_t R, int64_t ncols, int64_t n, int dt, int cus, TNPlan* P);

// Plain types with `fine` false, for a caller's workspace that does not hold
// those partials: at least eight steps per wavefront, two workgroups per CU.
void plan_tn_coarse(int64_t R, int64_t ncols, int64_t n, int dt, int cus, TNPlan* P) {
    P->pf = (int)env_int("TSM2X_TN_PF", 1);
    P->ct = ncols > 16 ? 2 : 1;
    P->groups = cdiv(cdiv(ncols, 16), P->ct) * P->ct;
    const int64_t RB = 16 * (16 / esize(dt)) * (P->ct == 2 ? 1 : 2);
    int64_t S = cdiv(2 * (int64_t)cus, P->groups / P->ct);
    if (S > R / (RB * 4 * 8)) S = R / (RB * 4 * 8);
    if (S < 1) S = 1;
    P->rslice = cdiv(cdiv(R, S), RB * 4) * (RB * 4);
    P->S = (int)cdiv(R, P->rslice);
    P->ws = P->S > 1 ? (size_t)P->groups * P->S * 256 * (n > 16 ? 2 : 1) * 8 : 0;
}

TNPlan plan_tn(int64_t R, int64_t ncols, int64_t n, int dt, int cus, bool fine = true) {
    TNPlan P{};
    if (plain_dtype(dt)) {
        fine ? plan_tn_plain(R, ncols, n, dt, cus, &P) : plan_tn_coarse(R, ncols, n, dt, cus, &P);
        return P;
    }
    // 16-bit forms.  Output tiles per workgroup: two share each Y tile when
    // there are several column groups (Y is then re-read by every group); they
    // take Y straight from L2 (staged in LDS too, two tiles needed one
    // workgroup per CU).  With n > 16 two tiles fit one workgroup per CU only;
    // with the next step in flight they still beat one tile (A 16384^2 and
    // 32768^2, n = 24, 32: split 3.4-4.2 -> 4.4-4.9 TB/s, single 2.0-2.6 ->
    // 2.5-3.1; without the prefetch one tile was faster)
    // bfloat16 planes with n <= 16 and more than four tiles: four tiles per
    // workgroup and one workgroup per CU on the 16-bit matrix cores
    // (tn_lp_kernel, MX; A 16384^2, n = 8: split 5.8 -> 6.6 TB/s, single
    // 5.4 -> 6.5 in the access-pattern probe of this grid)
    // For n > 16 the four tiles take Y's bf16 terms split once per call into
    // the workspace (their registers would not hold the split in the step;
    // A 16384^2, n = 32: split 4.4 -> 5.3 TB/s, single 3.4 -> 4.7), while
    // Y's terms stay below 256 MB (192 bytes per row: R up to 1.4 M).
    const bool bf = dt == DT_BF16 || dt == DT_BF16_SPLIT;
    const size_t yt_bytes = lp_bterms_bytes(R, n);
    const bool four = bf && cdiv(ncols, 16) > 4 && (n <= 16 || yt_bytes <= ((size_t)256 << 20));
    const int ct_dflt = four ? 4 : 2;
    P.ct = ncols > 16 ? (int)env_int("TSM2X_TN_CT", ct_dflt) : 1;
    if (P.ct == 4 && !bf) P.ct = 2;
    if (P.ct != 1 && P.ct != 2 && P.ct != 4) P.ct = 1;
    const int64_t RB = 128;                   // rows per wavefront step
    const int NT16 = n <= 16 ? 1 : 2;
    P.groups = cdiv(cdiv(ncols, 16), P.ct) * P.ct;
    const int64_t target = env_int("TSM2X_TN_TARGET_BLOCKS", (int64_t)cus * (P.ct == 4 ? 1 : 2));
    int64_t S = cdiv(target, P.groups / P.ct);
    const int64_t s_len = R / (RB * 4 * 8);   // >= 8 steps per wavefront
    if (S > s_len) S = s_len;
    if (S < 1) S = 1;
    int64_t rs = cdiv(R, S);
    rs = cdiv(rs, RB * 4) * (RB * 4);
    P.rslice = rs;
    P.S = (int)cdiv(R, rs);
    if (P.S < 1) P.S = 1;
    P.ws = P.S > 1 ? (size_t)P.groups * P.S * 256 * NT16 * 8 : 0;
    P.yt = P.ct == 4 && n > 16;
    if (P.yt) {
        P.yt_off = (P.ws + 255) / 256 * 256;
        P.ws = P.yt_off + yt_bytes;
    }
    // The next step held in flight (tn_lp_kernel), where it measured faster.
    // 16-bit single form: always (n = 8 and 16: 3.8-4.2 -> 4.8-5.7
    // TB/s) and for n > 16 (above).  16-bit split form with n <= 16, whose
    // steps move twice the bytes: only when the grid holds more than two
    // workgroups per CU (at A 16384^2, n = 8, one round of 512 workgroups:
    // 5.80 TB/s without, 5.21 with; at 32768^2, four rounds: 6.34 -> 6.51
    // (n = 8), 5.89 -> 6.17 (n = 16)).  bfloat16 planes with several column
    // groups run on the bf16 matrix cores (tn_lp_kernel, MX): with four tiles
    // the single form takes two steps (probe, A 16384^2, n = 8: 6.6 TB/s
    // against 5.8 with one; packed dC terms, n = 32: 4.7 against 3.8) and the
    // split form one (two do not fit its registers); with two tiles (an
    // override) one step for n <= 8 (5.5 against 4.9 TB/s).
    const bool split = dt == DT_BF16_SPLIT || dt == DT_F16_SPLIT;
    const bool mx = bf && (!split || n <= 16 || P.yt) && P.groups / P.ct > 1;
    const bool pf = mx ? P.ct == 4 || n > 8
                       : !split || n > 16 || (P.groups / P.ct) * P.S > 2 * (int64_t)cus;
    P.pf = (int)env_int("TSM2X_TN_PF", pf ? 1 : 0);
    return P;
}

void plan_tn_plain(int64_t R, int64_t ncols, int64_t n, int dt, int cus, TNPlan* P) {
    const bool wide = n > 16;
    const int es = esize(dt);
    P->pf = (int)env_int("TSM2X_TN_PF", 1);
    double best = 0;
    for (int ct = ncols > (wide ? 16 : 32) ? 2 : 1; ct >= (wide && ncols > 16 ? 2 : 1); --ct) {
        const int64_t RB = 16 * (16 / es) * (wide || ct == 2 ? 1 : 2);    // rows per wavefront step
        const int64_t gx = cdiv(cdiv(ncols, 16), ct);
        // the time of a split in bytes at the streaming rate: X (with one tile
        // Y is staged twice as often, 6 %), the second launch, 4 to 5 us with
        // what it costs the host, and the partials, written and read once
        // (one group reads the columns that there are, of two the last is
        // moved up and reads 16)
        const double bytes = (double)R * (gx == 1 ? ncols : gx * ct * 16) * es *
                             (wide || ct == 2 ? 1.0 : 1.06);
        const int64_t most = R / (RB * 4 * 2);
        int64_t last = 0;
        // candidates: one to four slices, and those that fill j workgroups per CU
        for (int64_t j = 0; j < 12; ++j) {
            int64_t S = j < 4 ? j + 1 : (j - 3) * cus / gx;
            if (S > most) S = most;
            if (S < 1) S = 1;
            if (S == last || (j >= 4 && S <= 4)) continue;
            last = S;
            const int64_t rs = cdiv(cdiv(R, S), RB * 4) * (RB * 4);
            const int64_t s = cdiv(R, rs);
            const double len = (double)rs / (RB * 4);
            double t = bytes * grid_time(gx * s, cus) * (len + 2) / len;
            // fewer columns than a workgroup takes: loads with bounds checks and
            // nothing held in flight, for which one workgroup per CU is too few
            // (1400000 x 6, n = 16: FP64 58 us with 249 workgroups, 47 with 498;
            // FP32 4000000 x 6, n = 1: 54 and 41)
            if (ncols < (wide ? 16 : 16 * ct) && gx * s <= cus) t *= 1.2;
            if (s > 1) t += 30e6 + (double)s * gx * ct * 16 * (wide ? 32 : 16) * 16;
            if (best == 0 || t < best) {
                best = t;
                P->ct = ct;
                P->groups = gx * ct;
                P->rslice = rs;
                P->S = (int)s;
            }
        }
    }
    P->ws = P->S > 1 ? (size_t)P->groups * P->S * 256 * (wide ? 2 : 1) * 8 : 0;
}

// A caller's workspace takes `need` bytes.
bool holds(const void* ws, size_t ws_bytes, size_t need) {
    return need == 0 || (ws_bytes >= need && ((uintptr_t)ws & 255u) == 0);
}

// Within its scope this thread may allocate and free although a stream is
// being captured.
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    const bool set = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
    ~RelaxedCapture() {
        if (set) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }
};

// Keeps a stream's buffer for one call: the launches that write and read the
// partials are enqueued with no other thread's between them.
struct WsHold {
    std::shared_ptr<WsBuf> buf;
    std::unique_lock<std::mutex> lock;
};

// The stream's entry of the table, locked.  The table is bounded: beyond
// kMaxWsBufs streams the one longest unused gives its buffer back (hipFree
// waits for the work on it), unless a graph may hold it.
hipError_t hold_buf(hipStream_t st, bool capturing, WsHold* h) {
    static thread_local char tag;
    const WsKey key(st, st == hipStreamPerThread ? &tag : nullptr);
    for (;;) {
        std::shared_ptr<WsBuf> old;
        {
            std::lock_guard<std::mutex> lk(g_mu);
            DevState* d = dev_state(nullptr);
            if (!d) return hipErrorInvalidDevice;
            std::shared_ptr<WsBuf>& e = d->bufs[key];
            if (!e) e = std::make_shared<WsBuf>();
            e->used = ++d->clock;
            h->buf = e;
            if (d->bufs.size() > kMaxWsBufs && !capturing) {
                auto lru = d->bufs.end();
                for (auto it = d->bufs.begin(); it != d->bufs.end(); ++it)
                    if (it->second != e && (lru == d->bufs.end() || it->second->used < lru->second->used)) {
                        std::unique_lock<std::mutex> l(it->second->mu, std::try_to_lock);
                        if (l && !it->second->captured) lru = it;
                    }
                if (lru != d->bufs.end()) {
                    std::unique_lock<std::mutex> l(lru->second->mu, std::try_to_lock);
                    if (l && !lru->second->captured) {
                        old = lru->second;
                        old->dead = true;
                        d->bufs.erase(lru);
                    }
                }
            }
        }
        if (old && old->p) {
            RelaxedCapture relaxed;
            (void)hipFree(old->p);
        }
        h->lock = std::unique_lock<std::mutex>(h->buf->mu);
        if (!h->buf->dead) return hipSuccess;
        h->lock.unlock();
    }
}

// Workspace: caller's (checked) or the library's buffer of the stream, which
// grows as calls need it.  A buffer that a captured launch was given is never
// freed before tsm2x_finalize, as a graph may hold its address: outgrown, it
// is retired, and its successor has at least twice its size, so that the
// retired ones together take no more than the one in use.
int get_ws(size_t need, void* user, size_t user_bytes, hipStream_t st, WsHold* h, void** out) try {
    *out = nullptr;
    if (need == 0) return TSM_SUCCESS;
    if (user) {
        if (!holds(user, user_bytes, need)) return TSM_ERR_WORKSPACE;
        *out = user;
        return TSM_SUCCESS;
    }
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;     // the null stream is never captured
    if (st && hipStreamIsCapturing(st, &cap) != hipSuccess) (void)hipGetLastError();
    const bool capturing = cap != hipStreamCaptureStatusNone;
    hipError_t e = hold_buf(st, capturing, h);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    WsBuf& b = *h->buf;
    if (b.bytes < need) {
        RelaxedCapture relaxed;
        size_t bytes = need < ((size_t)1 << 20) ? ((size_t)1 << 20) : need;
        const size_t twice = b.captured && 2 * b.bytes > bytes ? 2 * b.bytes : bytes;
        if (b.p && (b.captured || capturing)) {
            std::lock_guard<std::mutex> lk(g_mu);
            if (DevState* d = dev_state(nullptr)) d->retired.push_back(b.p);
        } else if (b.p) {
            e = hipFree(b.p);
        }
        b.p = nullptr;
        b.bytes = 0;
        b.captured = false;
        if (e != hipSuccess) return hip_fail(e, "hipFree(workspace)");
        e = hipMalloc(&b.p, twice);
        if (e == hipSuccess) {
            bytes = twice;
        } else if (twice > bytes) {
            (void)hipGetLastError();
            e = hipMalloc(&b.p, bytes);
        }
        if (e != hipSuccess) {
            b.p = nullptr;
            g_last_hip = std::string("hipMalloc(workspace): ") + hipGetErrorString(e);
            return TSM_ERR_ALLOC;
        }
        b.bytes = bytes;
    }
    b.captured |= capturing;
    *out = b.p;
    return TSM_SUCCESS;
} catch (const std::bad_alloc&) {
    return TSM_ERR_ALLOC;
}

// Validation of (m, k, n, A, lda, B, ldb, C, ldc, dtype) for C = A*B with
// column-major (or, for `rowA`, row-major) A.  `base` is the position of m.
int check_mm(int base, int64_t m, int64_t k, int64_t n, const void* A, int64_t lda,
             const void* B, int64_t ldb, const void* C, int64_t ldc, int dtype, bool rowA) {
    if (m < 0) return -(base + 0);
    if (k < 0) return -(base + 1);
    if (n < 0) return -(base + 2);
    if (!A && m > 0 && k > 0) return -(base + 3);
    const int64_t mina = rowA ? (k > 1 ? k : 1) : (m > 1 ? m : 1);
    if (lda < mina) return -(base + 4);
    if (!B && k > 0 && n > 0) return -(base + 5);
    if (ldb < (k > 1 ? k : 1)) return -(base + 6);
    if (!C && m > 0 && n > 0) return -(base + 7);
    if (ldc < (m > 1 ? m : 1)) return -(base + 8);
    if (!valid_dtype(dtype)) return -(base + 9);
    return TSM_SUCCESS;
}

// Validation for the extended product entry points; argument positions
// 1 transA, 2 transB, 3 m, 4 k, 5 n, 6 A, 7 lda, 8 B, 9 ldb, 10 beta, 11 C,
// 12 ldc, 13 dtype.
int check_ex(int transA, int transB, int64_t m, int64_t k, int64_t n, const void* A,
             int64_t lda, const void* B, int64_t ldb, const void* C, int64_t ldc, int dtype) {
    if (transA != 0 && transA != 1) return -1;
    if (transB != 0 && transB != 1) return -2;
    if (m < 0) return -3;
    if (k < 0) return -4;
    if (n < 0) return -5;
    if (!A && m > 0 && k > 0) return -6;
    const int64_t mina = transA ? k : m;
    if (lda < (mina > 1 ? mina : 1)) return -7;
    if (!B && k > 0 && n > 0) return -8;
    const int64_t minb = transB ? n : k;
    if (ldb < (minb > 1 ? minb : 1)) return -9;
    if (!C && m > 0 && n > 0) return -11;
    if (ldc < (m > 1 ? m : 1)) return -12;
    if (!valid_dtype(dtype)) return -13;
    return TSM_SUCCESS;
}

// Leading dimension of the column-major copy of a transposed B (k x n), kept
// a multiple of 16 bytes so the kernels' 16-byte B loads apply.
int64_t bt_ld(int64_t k, int ce) { return cdiv(k, 16 / ce) * (16 / ce); }

// Bytes of split partials of a TSM2R-kernel product of at most 32 columns,
// for the kernel instance the call launches (`vec`: A is aligned()); `fine` as
// in the planners.
size_t tsm2r_part(int transA, int64_t m, int64_t k, int64_t n, int dtype, bool vec, bool fine) {
    const int cus = cu_count();
    if (!plain_dtype(dtype)) {
        NNPlan P{};
        plan_tsm2r_lp(m, k, n, dtype, cus, vec, &P, fine);
        return P.ws;
    }
    if (transA) return plan_tn(k, m, n, dtype, cus, fine).ws;
    NNPlan P{};
    return plan_nn(m, k, n, dtype, cus, vec, &P, fine) ? 0 : P.ws;
}

// What follows the partials: room for B when it is given transposed (plain
// types), or for B's packed 16-bit terms (precision form, B read in either
// order).
size_t behind_part(int64_t k, int64_t n, int dtype, bool transB) {
    if (!plain_dtype(dtype)) return lp_bterms_bytes(k, n);
    return transB ? (size_t)bt_ld(k, esize(dtype)) * n * esize(dtype) : 0;
}

// Workspace of a panel of a TSM2R-kernel product.
size_t tsm2r_ws(int transA, int64_t m, int64_t k, int64_t n, int dtype, bool transB, bool vec,
                bool fine = true) {
    return align256(tsm2r_part(transA, m, k, n, dtype, vec, fine)) + behind_part(k, n, dtype, transB);
}

// A column-major A of at most 32 rows, wider than the TSM2L kernels take:
// both operands are long in k and short otherwise (tsmttsm of row-major
// matrices), which the tt kernel reads as they stand; the TSM2R kernel tiles
// rows, of which there are few here (16 x 1048576, n = 16, B row-major: FP32
// 105 us, tt 28, FP64 86 and 48; B column-major: 101 and 30, 86 and 54).
// A plan pinned for the shape keeps the TSM2R kernel.
bool tt_shape(int transA, int64_t m, int64_t k, int64_t n, int dtype) {
    if (transA || m > 32 || k <= 32 || !plain_dtype(dtype)) return false;
    const NNPin pin = pin_of(m, k, n, dtype);
    return pin.S == 0 && pin.tall < 0;
}

// The most any plan of the call can need (the query does not know A's
// alignment, which picks the kernel instance).
size_t tsm2r_ws_max(int transA, int64_t m, int64_t k, int64_t n, int dtype, bool transB) {
    const size_t a = tsm2r_ws(transA, m, k, n, dtype, transB, true);
    const size_t b = tsm2r_ws(transA, m, k, n, dtype, transB, false);
    const size_t c = tt_shape(transA, m, k, n, dtype) ? tt_ws(k, (int)m, (int)n, cu_count()) : 0;
    return a > b ? (a > c ? a : c) : (b > c ? b : c);
}

// Columns of B and C per pass over A.  A column-major A on the TSM2R kernel
// takes 64: with two passes of 32 the second reads A again, and the kernel is
// bound by the matrix cores at 64 (20480^2, n = 64: FP64 1270 us in two
// passes, 918 in one, FP32 590 and 501; n = 33: 1109 and 685, 544 and 377).  32 elsewhere, for a caller's workspace that holds
// the partials of 32 columns only, and where a plan of a narrower panel is
// pinned.  Also for a tall A of few columns, where a wavefront has too few
// steps to gain back what its fewer neighbours cost: FP64 beyond 48 columns
// (1000000 x 64, n = 64: 523 us in one pass, 396 in two; 50000 x 90: 48 and 40;
// but 300000 x 72: 149 and 169), FP32 where the wavefronts' 16-column chunks are not
// whole (1000000 x 40, n = 48: 347 and 271; 50000 x 40 one pass is the faster).
int64_t panel_width(bool lform, int transA, int transB, int64_t m, int64_t k, int64_t n,
                    const void* A, int64_t lda, int dtype, const void* ws, size_t ws_bytes) {
    if (n <= 32 || transA || !plain_dtype(dtype) || (lform && k <= 32) || m <= 32) return 32;
    auto pinned = [&](int64_t w) {
        const NNPin p = pin_of(m, k, w, dtype);
        return p.S > 0 || p.tall >= 0;
    };
    if (pinned(32) || (n % 32 && pinned(n % 32))) return 32;
    if (dtype == TSM_F64 ? n > 48 && (k <= 68 || k > 80) && k <= 96 && m >= 1 << 15
                         : k <= 96 && k % 16 != 0 && m >= 1 << 18)
        return 32;
    if (ws && !holds(ws, ws_bytes, tsm2r_ws(0, m, k, n < 64 ? n : 64, dtype, transB,
                                            aligned(A, lda, dtype, m, k, n))))
        return 32;
    return 64;
}

// Bytes a caller's workspace must have for a product of n columns in panels
// of panel_width: those of the finer or the coarser split, whichever is less.
size_t caller_ws(bool lform, int transA, int transB, int64_t m, int64_t k, int64_t n,
                 const void* A, int64_t lda, int dtype, const void* ws, size_t ws_bytes) {
    if (lform && !transA && k <= 32) return 0;
    const int64_t panel = panel_width(lform, transA, transB, m, k, n, A, lda, dtype, ws, ws_bytes);
    size_t most = 0;
    for (const int64_t w : {n < panel ? n : panel, n > panel ? n % panel : (int64_t)0}) {
        if (w == 0) continue;
        const bool al = (transA && k <= 32) || aligned(A, lda, dtype, m, k, w);
        const size_t fine = tsm2r_ws(transA, m, k, w, dtype, transB, al);
        const size_t coarse = tsm2r_ws(transA, m, k, w, dtype, transB, al, false);
        const size_t b = fine < coarse ? fine : coarse;
        if (b > most) most = b;
    }
    return most;
}

// C := beta*C + op(A)*op(B) on validated arguments.  `lform` asks for the TSM2L
// kernels (all of B on chip) for a column-major A with k <= 32; other shapes
// run on the TSM2R kernels, which are correct for any k.  A row-major A with
// k <= 32 takes the TSM2L kernel either way: the reduction kernel splits the
// contiguous dimension over its lanes and wavefronts, and one of at most 32
// elements leaves most of them idle (FP32 4194304 x 16, n = 16: 1499 us
// there, 105 here; 17 columns, n = 28: 2.1 ms and 158 us; a column-major A
// takes 103 and 152).  More
// columns than one pass takes (panel_width) run in panels of B and C, A being
// read once per panel.
int product(bool lform, int transA, int transB, int64_t m, int64_t k, int64_t n, const void* A,
            int64_t lda, const void* B, int64_t ldb, double beta, void* C, int64_t ldc,
            int dtype, void* ws, size_t ws_bytes, hipStream_t st) {
    if (transA && !plain_dtype(dtype)) return TSM_ERR_UNSUPPORTED;   // planes are column-major
    if (m == 0 || n == 0) return TSM_SUCCESS;
    const int ce = plain_dtype(dtype) ? esize(dtype) : 4;             // element size of B, C
    const int cdt = plain_dtype(dtype) ? dtype : TSM_F32;
    if (k == 0) {
        launch_fill_scale(m, n, C, ldc, beta, cdt, st);
        return check_launch("fill_scale_kernel");
    }
    const int64_t panel = panel_width(lform, transA, transB, m, k, n, A, lda, dtype, ws, ws_bytes);
    if (n > panel) {
        // no panel runs if the caller's workspace is too small for any of them
        for (const int64_t w : {panel, n % panel})
            if (ws && w > 0 &&
                !holds(ws, ws_bytes, caller_ws(lform, transA, transB, m, k, w, A, lda, dtype, ws, ws_bytes)))
                return TSM_ERR_WORKSPACE;
        for (int64_t p0 = 0; p0 < n; p0 += panel) {
            const int64_t np = n - p0 < panel ? n - p0 : panel;
            const char* Bp = (const char*)B + (transB ? p0 : p0 * ldb) * ce;
            char* Cp = (char*)C + p0 * ldc * ce;
            int rc = product(lform, transA, transB, m, k, np, A, lda, Bp, ldb, beta, Cp, ldc,
                             dtype, ws, ws_bytes, st);
            if (rc) return rc;
        }
        return TSM_SUCCESS;
    }
    const int cus = cu_count();
    const bool rowx = transA && k <= 32;      // plain types only (above)
    if (rowx && ws) {
        // nothing is put there, but a workspace that this product's size
        // query would not have given is refused all the same
        if (!holds(ws, ws_bytes, tsm2r_ws(transA, m, k, n, dtype, transB, true)))
            return TSM_ERR_WORKSPACE;
    }
    if ((lform && !transA && k <= 32) || rowx) {
        // B(j, p) at B[j*bsj + p*bsp]: both orders of B are plain strides here
        const int64_t bsj = transB ? ldb : 1, bsp = transB ? 1 : ldb;
        if (!plain_dtype(dtype)) {
            launch_tsm2l_lp(m, k, n, A, lda, (const float*)B, bsj, bsp, (float)beta, (float*)C,
                            ldc, dtype, cus, st);
            return check_launch("tsm2l_lp_kernel");
        }
        RTPlan P = plan_rowtile(m, k, n, dtype, cus);
        LaunchRT L{};
        L.m = m; L.kin = (int)k; L.nout = n; L.X = A; L.ldx = lda; L.Y = B; L.ys_in = bsj;
        L.x_rowmajor = rowx;
        L.ys_out = bsp; L.O = C; L.ldo = ldc; L.kp = P.kp; L.cols_per_block = (int)P.cpb;
        L.blocks_x = P.bx; L.blocks_y = P.by; L.cus = cus; L.beta = beta;
        if (launch_rowtile(L, dtype, st)) return TSM_ERR_UNSUPPORTED;
        return check_launch("rowtile_kernel");
    }
    WsHold hold;
    if (tt_shape(transA, m, k, n, dtype)) {
        // a caller's workspace of the size the TSM2R kernels need is accepted,
        // and they run if it is too small for this kernel's partials
        const size_t need = tt_ws(k, (int)m, (int)n, cus);
        const size_t nn = tsm2r_ws(transA, m, k, n, dtype, transB, true);
        if (!ws || holds(ws, ws_bytes, nn > need ? nn : need)) {
            void* w = nullptr;
            const int rc = get_ws(need, ws, ws_bytes, st, &hold, &w);
            if (rc) return rc;
            LaunchTT L{};
            L.R = k; L.ma = (int)m; L.n = (int)n; L.X = A; L.ldx = lda; L.Y = B; L.ldy = ldb;
            L.y_rowmajor = transB; L.O = C; L.ldo = ldc; L.part = (double*)w; L.beta = beta;
            L.cus = cus;
            if (launch_tt(L, dtype, st)) return TSM_ERR_UNSUPPORTED;
            return check_launch("tt_kernel");
        }
    }
    // TSM2R kernels; workspace = [split partials][B copied column-major, or
    // B's packed 16-bit terms for the precision form]
    const bool avec = aligned(A, lda, dtype, m, k, n);
    // The reduction kernel reads B in runs down its columns.  A row-major B of
    // up to 16 columns it loads value by value, which takes less than the copy
    // and its launch, where a wavefront has up to 256 rows of it (1024^2, n = 4:
    // FP32 10.2 us and 11.4 with the copy, FP64 9.0 and 11.4; FP64 2048^2, n = 16,
    // 128 rows: 12.2 and 14.6; but FP32 1448^2, n = 4, 384 rows: 14.6 and 11.4;
    // 2048^2, 512: 18.1 and 11.6; FP64 1448^2, 384 rows: n = 4 10.5 and 11.5, n =
    // 8 14.3 and 11.5) and the workgroups' rows come to no more than 256 on a CU
    // (FP32 8192 x 256, n = 16, 64 rows in 256 workgroups: 7.7 and 11.5; 15808 x
    // 784, n = 16, 256 in 988: 43 and 39; 65536 x 128, 64 in 2048: 16.7 and 15.5).
    bool direct = plain_dtype(dtype) && transB && !transA;
    NNPlan P{};
    TNPlan T{};
    size_t part = 0, need = 0;               // the partials' bytes, and with what follows them
    auto plan = [&](bool fine) {
        if (!plain_dtype(dtype)) {
            plan_tsm2r_lp(m, k, n, dtype, cus, avec, &P, fine);
        } else if (transA) {
            T = plan_tn(k, m, n, dtype, cus, fine);
            const int64_t rows = T.rslice / 4 < k ? T.rslice / 4 : k;
            direct = transB && n <= 16 && rows <= (dtype == TSM_F64 && n <= 4 ? 384 : 256) &&
                     T.groups / T.ct * T.S * rows <= 256 * (int64_t)cus;
        } else if (plan_nn(m, k, n, dtype, cus, avec, &P, fine)) {
            return false;
        }
        part = align256(transA ? T.ws : P.ws);
        need = part + behind_part(k, n, dtype, transB && (ws || !direct));
        return true;
    };
    if (!plan(true)) return TSM_ERR_UNSUPPORTED;
    if (ws && !holds(ws, ws_bytes, need) && !plan(false)) return TSM_ERR_UNSUPPORTED;
    void* w = nullptr;
    int rc = get_ws(need, ws, ws_bytes, st, &hold, &w);
    if (rc) return rc;
    if (!plain_dtype(dtype)) {
        // A: 16-bit hi plane (and lo plane lda*k elements after it); B, C float
        void* bt = (char*)w + part;
        launch_split_b(k, n, (const float*)B, transB ? ldb : 1, transB ? 1 : ldb, dtype, bt, st);
        rc = check_launch("split_b_kernel");
        if (rc) return rc;
        LaunchNN L{};
        L.fn = P.fn;
        L.m = m; L.k = k; L.n = n; L.A = A; L.lda = lda; L.B = bt; L.ldb = 0; L.C = C;
        L.ldc = ldc; L.np = P.np; L.tile_rows = P.tile_rows; L.tiles = P.tiles; L.S = P.S;
        L.kslice = P.kslice; L.beta = beta;
        if (P.S > 1) L.part = (double*)w;
        launch_tsm2r_lp(L, dtype, st);
        return check_launch("tsm2r_lp_kernel");
    }
    const void* Bk = B;
    int64_t ldbk = ldb;
    const bool copy = transB && !direct;
    if (copy) {
        void* bc = (char*)w + part;
        launch_transpose(k, n, B, ldb, bc, bt_ld(k, ce), cdt, st);
        rc = check_launch("transpose_kernel");
        if (rc) return rc;
        Bk = bc;
        ldbk = bt_ld(k, ce);
    }
    if (transA) {
        // A given transposed is the column-major k x m matrix X = A^T (ld lda):
        // C = X^T * B, a reduction along the contiguous dimension.
        LaunchTN L{};
        L.R = k; L.ncols = m; L.n = n;
        L.X = A; L.ldx = lda; L.Y = Bk; L.ldy = ldbk; L.O = C; L.ldo = ldc;
        L.y_rowmajor = transB && !copy;
        L.groups = T.groups; L.S = T.S; L.rslice = T.rslice; L.ct = T.ct;
        L.pf = T.pf;
        L.beta = beta;
        if (T.S > 1) L.part = (double*)w;
        if (launch_tn(L, dtype, st)) return TSM_ERR_UNSUPPORTED;
        return check_launch("tn_kernel");
    }
    LaunchNN L{};
    L.fn = transB ? P.fn_bt : P.fn;
    L.m = m; L.k = k; L.n = n; L.A = A; L.lda = lda; L.B = Bk; L.ldb = ldbk; L.C = C; L.ldc = ldc;
    L.np = P.np; L.tile_rows = P.tile_rows; L.tiles = P.tiles; L.S = P.S; L.kslice = P.kslice;
    L.beta = beta;
    L.pf = P.pf;
    if (P.S > 1) L.part = (double*)w;
    if (launch_tsm2r_nn(L, dtype, st)) return TSM_ERR_UNSUPPORTED;
    return check_launch("tsm2r_nn_kernel");
}

}  // namespace

extern "C" {

int tsm2r_ex(int transA, int transB, int64_t m, int64_t k, int64_t n, const void* A,
             int64_t lda, const void* B, int64_t ldb, double beta, void* C, int64_t ldc,
             int dtype, void* ws, size_t ws_bytes, void* stream) {
    int rc = check_ex(transA, transB, m, k, n, A, lda, B, ldb, C, ldc, dtype);
    if (rc) return rc;
    return product(false, transA, transB, m, k, n, A, lda, B, ldb, beta, C, ldc, dtype, ws,
                   ws_bytes, (hipStream_t)stream);
}

int tsm2l_ex(int transA, int transB, int64_t m, int64_t k, int64_t n, const void* A,
             int64_t lda, const void* B, int64_t ldb, double beta, void* C, int64_t ldc,
             int dtype, void* ws, size_t ws_bytes, void* stream) {
    int rc = check_ex(transA, transB, m, k, n, A, lda, B, ldb, C, ldc, dtype);
    if (rc) return rc;
    return product(true, transA, transB, m, k, n, A, lda, B, ldb, beta, C, ldc, dtype, ws,
                   ws_bytes, (hipStream_t)stream);
}

int tsm2x_gemm(int transA, int transB, int64_t m, int64_t k, int64_t n, const void* A,
               int64_t lda, const void* B, int64_t ldb, double beta, void* C, int64_t ldc,
               int dtype, void* ws, size_t ws_bytes, void* stream) {
    int rc = check_ex(transA, transB, m, k, n, A, lda, B, ldb, C, ldc, dtype);
    if (rc) return rc;
    // the paper's two shape classes: a tall-and-skinny A (k small, all of B on
    // chip) goes to TSM2L, a large A to TSM2R
    const bool lform = transA == 0 && k <= 32;
    return product(lform, transA, transB, m, k, n, A, lda, B, ldb, beta, C, ldc, dtype, ws,
                   ws_bytes, (hipStream_t)stream);
}

int tsm2r(int64_t m, int64_t k, int64_t n, const void* A, int64_t lda, const void* B,
          int64_t ldb, void* C, int64_t ldc, int dtype, void* stream) {
    int rc = check_mm(1, m, k, n, A, lda, B, ldb, C, ldc, dtype, false);
    if (rc) return rc;
    return product(false, 0, 0, m, k, n, A, lda, B, ldb, 0.0, C, ldc, dtype, nullptr, 0,
                   (hipStream_t)stream);
}

int tsm2l(int64_t m, int64_t k, int64_t n, const void* A, int64_t lda, const void* B,
          int64_t ldb, void* C, int64_t ldc, int dtype, void* stream) {
    int rc = check_mm(1, m, k, n, A, lda, B, ldb, C, ldc, dtype, false);
    if (rc) return rc;
    return product(true, 0, 0, m, k, n, A, lda, B, ldb, 0.0, C, ldc, dtype, nullptr, 0,
                   (hipStream_t)stream);
}

// tsm_grad_a on B(j, p) = B[j*bsj + p*bsp], arguments checked
static int run_grad_a(int64_t m, int64_t k, int64_t n, const void* dC, int64_t lddc, const void* B,
                      int64_t bsj, int64_t bsp, void* dA, int64_t ldda, int dtype, hipStream_t st) {
    if (n > 32 || !plain_dtype(dtype)) return TSM_ERR_UNSUPPORTED;
    if (m == 0 || k == 0) return TSM_SUCCESS;
    if (n == 0) {
        launch_fill_scale(m, k, dA, ldda, 0.0, dtype, st);
        return check_launch("fill_scale_kernel");
    }
    // dA = dC * B^T: X = dC (m x n), Y(p, j) = B(j, p)
    RTPlan P = plan_rowtile(m, n, k, dtype, cu_count());
    LaunchRT L{};
    L.m = m; L.kin = (int)n; L.nout = k; L.X = dC; L.ldx = lddc; L.Y = B; L.ys_in = bsp;
    L.ys_out = bsj; L.O = dA; L.ldo = ldda; L.kp = P.kp; L.cols_per_block = (int)P.cpb;
    L.blocks_x = P.bx; L.blocks_y = P.by; L.cus = cu_count();
    if (launch_rowtile(L, dtype, st)) return TSM_ERR_UNSUPPORTED;
    return check_launch("rowtile_kernel");
}

int tsm_grad_a_ex(int transB, int64_t m, int64_t k, int64_t n, const void* dC, int64_t lddc,
                  const void* B, int64_t ldb, void* dA, int64_t ldda, int dtype, void* stream) {
    if (transB != 0 && transB != 1) return -1;
    if (m < 0) return -2;
    if (k < 0) return -3;
    if (n < 0) return -4;
    if (!dC && m > 0 && n > 0) return -5;
    if (lddc < (m > 1 ? m : 1)) return -6;
    if (!B && k > 0 && n > 0) return -7;
    if (ldb < ((transB ? n : k) > 1 ? (transB ? n : k) : 1)) return -8;
    if (!dA && m > 0 && k > 0) return -9;
    if (ldda < (m > 1 ? m : 1)) return -10;
    if (!valid_dtype(dtype)) return -11;
    return run_grad_a(m, k, n, dC, lddc, B, transB ? ldb : 1, transB ? 1 : ldb, dA, ldda, dtype,
                      (hipStream_t)stream);
}

int tsm_grad_a(int64_t m, int64_t k, int64_t n, const void* dC, int64_t lddc, const void* B,
               int64_t ldb, void* dA, int64_t ldda, int dtype, void* stream) {
    if (m < 0) return -1;
    if (k < 0) return -2;
    if (n < 0) return -3;
    if (!dC && m > 0 && n > 0) return -4;
    if (lddc < (m > 1 ? m : 1)) return -5;
    if (!B && k > 0 && n > 0) return -6;
    if (ldb < (k > 1 ? k : 1)) return -7;
    if (!dA && m > 0 && k > 0) return -8;
    if (ldda < (m > 1 ? m : 1)) return -9;
    if (!valid_dtype(dtype)) return -10;
    return run_grad_a(m, k, n, dC, lddc, B, 1, ldb, dA, ldda, dtype, (hipStream_t)stream);
}

int tsm_grad_b(int64_t m, int64_t k, int64_t n, const void* A, int64_t lda, const void* dC,
               int64_t lddc, void* dB, int64_t lddb, int dtype, void* ws, size_t ws_bytes,
               void* stream) {
    if (m < 0) return -1;
    if (k < 0) return -2;
    if (n < 0) return -3;
    if (!A && m > 0 && k > 0) return -4;
    if (lda < (m > 1 ? m : 1)) return -5;
    if (!dC && m > 0 && n > 0) return -6;
    if (lddc < (m > 1 ? m : 1)) return -7;
    if (!dB && k > 0 && n > 0) return -8;
    if (lddb < (k > 1 ? k : 1)) return -9;
    if (!valid_dtype(dtype)) return -10;
    if (n > 32) return TSM_ERR_UNSUPPORTED;
    if (k == 0 || n == 0) return TSM_SUCCESS;
    hipStream_t st = (hipStream_t)stream;
    if (m == 0) {
        launch_fill_scale(k, n, dB, lddb, 0.0, plain_dtype(dtype) ? dtype : TSM_F32, st);
        return check_launch("fill_scale_kernel");
    }
    // dB = A^T * dC: X = A (R = m rows, k columns), Y = dC.
    TNPlan P = plan_tn(m, k, n, dtype, cu_count());
    if (ws && !holds(ws, ws_bytes, P.ws)) P = plan_tn(m, k, n, dtype, cu_count(), false);
    void* w = nullptr;
    WsHold hold;
    int rc = get_ws(P.ws, ws, ws_bytes, st, &hold, &w);
    if (rc) return rc;
    LaunchTN L{};
    L.R = m; L.ncols = k; L.n = n; L.X = A; L.ldx = lda; L.Y = dC; L.ldy = lddc; L.O = dB;
    L.ldo = lddb; L.groups = P.groups; L.S = P.S; L.rslice = P.rslice; L.ct = P.ct;
    L.pf = P.pf;
    if (P.S > 1) L.part = (double*)w;
    if (P.yt) L.yt = (char*)w + P.yt_off;
    if (!plain_dtype(dtype)) {
        if (launch_tn_lp(L, dtype, st)) return TSM_ERR_UNSUPPORTED;
        return check_launch("tn_lp_kernel");
    }
    if (launch_tn(L, dtype, st)) return TSM_ERR_UNSUPPORTED;
    return check_launch("tn_kernel");
}

}  // extern "C"

// Scratch of the allocation-free fused backward: room for the dB partials
// of 2048 workgroups of the widest instance (32 x 32 doubles each), i.e. a
// persistent grid of 8 resident workgroups on each of 256 compute units.
// Every device holds its own copy for the life of the process.  Host code
// never passes `scratch` itself (on the host the name is only a stand-in);
// it uses the per-device address hipGetSymbolAddress returns.
static constexpr size_t kBwdScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) double scratch[kBwdScratchBytes / sizeof(double)];

namespace {

// Argument checks of tsm2l_backward (positions 1..14).
int check_bwd(int64_t m, int64_t k, int64_t n, const void* A, int64_t lda, const void* B,
              int64_t ldb, int64_t minb, const void* dC, int64_t lddc, const void* dA, int64_t ldda,
              const void* dB, int64_t lddb, int dtype) {
    if (m < 0) return -1;
    if (k < 0) return -2;
    if (n < 0) return -3;
    if (!A && m > 0 && k > 0) return -4;
    if (lda < (m > 1 ? m : 1)) return -5;
    if (!B && k > 0 && n > 0) return -6;
    if (ldb < (minb > 1 ? minb : 1)) return -7;
    if (!dC && m > 0 && n > 0) return -8;
    if (lddc < (m > 1 ? m : 1)) return -9;
    if (!dA && m > 0 && k > 0) return -10;
    if (ldda < (m > 1 ? m : 1)) return -11;
    if (!dB && k > 0 && n > 0) return -12;
    if (lddb < (k > 1 ? k : 1)) return -13;
    if (!valid_dtype(dtype)) return -14;
    if (k > 32 || n > 32) return TSM_ERR_UNSUPPORTED;
    return TSM_SUCCESS;
}

// The fused backward on checked arguments; `part` supplies the dB partials
// (one k x n double block per workgroup): part(need) returns the buffer for
// `need` bytes, or null with *rc set.
template <typename PartFn>
int run_bwd(int64_t m, int64_t k, int64_t n, const void* A, int64_t lda, const void* B,
            int64_t bsj, int64_t bsp, const void* dC, int64_t lddc, void* dA, int64_t ldda, void* dB,
            int64_t lddb, int dtype, hipStream_t st, PartFn part) {
    if (k == 0) return TSM_SUCCESS;
    const int odt = plain_dtype(dtype) ? dtype : TSM_F32;      // B, dC, dA, dB
    if (m == 0 || n == 0) {
        // dA (m x k) is zero when n == 0; dB (k x n) is zero when m == 0
        if (m > 0) launch_fill_scale(m, k, dA, ldda, 0.0, odt, st);
        if (n > 0) launch_fill_scale(k, n, dB, lddb, 0.0, odt, st);
        return check_launch("fill_scale_kernel");
    }
    LaunchBwd L{};
    L.m = m; L.k = k; L.n = n; L.A = A; L.lda = lda; L.B = B; L.bsj = bsj; L.bsp = bsp; L.dC = dC;
    L.lddc = lddc; L.dA = dA; L.ldda = ldda; L.dB = dB; L.lddb = lddb; L.cus = cu_count();
    int64_t blocks = 0;
    launch_tsm2l_bwd(L, dtype, &blocks, st, true);
    const size_t need = (size_t)blocks * (k <= 16 ? 16 : 32) * (n <= 16 ? 16 : 32) * 8;
    int rc = TSM_SUCCESS;
    L.part = (double*)part(need, &rc);
    if (rc) return rc;
    launch_tsm2l_bwd(L, dtype, &blocks, st, false);
    return check_launch("tsm2l_bwd_kernel");
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices] = {};

// This device's scratch address (looked up once per device, with the device
// current); null with *rc set on failure.
void* scratch_ptr(int* rc) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        *rc = hip_fail(e, "hipGetDevice");
        return nullptr;
    }
    if (dev < 0 || dev >= kMaxDevices) {
        g_last_hip = "scratch: device index beyond the supported 64 devices";
        *rc = TSM_ERR_UNSUPPORTED;
        return nullptr;
    }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            *rc = hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol,
                           "hipGetSymbolAddress(scratch)");
            return nullptr;
        }
        g_scratch[dev] = p;
    }
    return g_scratch[dev];
}

}  // namespace

extern "C" {

int tsm2l_backward_noalloc(int64_t m, int64_t k, int64_t n, const void* A, int64_t lda,
                           const void* B, int64_t ldb, const void* dC, int64_t lddc, void* dA,
                           int64_t ldda, void* dB, int64_t lddb, int dtype, void* stream) {
    int rc = check_bwd(m, k, n, A, lda, B, ldb, k, dC, lddc, dA, ldda, dB, lddb, dtype);
    if (rc) return rc;
    return run_bwd(m, k, n, A, lda, B, 1, ldb, dC, lddc, dA, ldda, dB, lddb, dtype,
                   (hipStream_t)stream, [](size_t need, int* prc) -> void* {
                       if (need > kBwdScratchBytes) {
                           g_last_hip = "tsm2l_backward_noalloc: the dB partials need " +
                                        std::to_string(need) + " bytes, beyond the " +
                                        std::to_string(kBwdScratchBytes) + "-byte scratch";
                           *prc = TSM_ERR_WORKSPACE;
                           return nullptr;
                       }
                       return scratch_ptr(prc);
                   });
}

int tsm2l_backward_ex(int transB, int64_t m, int64_t k, int64_t n, const void* A, int64_t lda,
                      const void* B, int64_t ldb, const void* dC, int64_t lddc, void* dA,
                      int64_t ldda, void* dB, int64_t lddb, int dtype, void* ws, size_t ws_bytes,
                      void* stream) {
    if (transB != 0 && transB != 1) return -1;
    const int rc = check_bwd(m, k, n, A, lda, B, ldb, transB ? n : k, dC, lddc, dA, ldda, dB, lddb,
                             dtype);
    if (rc) return rc < 0 ? rc - 1 : rc;
    WsHold hold;
    return run_bwd(m, k, n, A, lda, B, transB ? ldb : 1, transB ? 1 : ldb, dC, lddc, dA, ldda, dB,
                   lddb, dtype, (hipStream_t)stream, [&](size_t need, int* prc) -> void* {
                       void* w = nullptr;
                       *prc = get_ws(need, ws, ws_bytes, (hipStream_t)stream, &hold, &w);
                       return w;
                   });
}

int tsm2l_backward(int64_t m, int64_t k, int64_t n, const void* A, int64_t lda, const void* B,
                   int64_t ldb, const void* dC, int64_t lddc, void* dA, int64_t ldda, void* dB,
                   int64_t lddb, int dtype, void* ws, size_t ws_bytes, void* stream) {
    int rc = check_bwd(m, k, n, A, lda, B, ldb, k, dC, lddc, dA, ldda, dB, lddb, dtype);
    if (rc) return rc;
    WsHold hold;
    return run_bwd(m, k, n, A, lda, B, 1, ldb, dC, lddc, dA, ldda, dB, lddb, dtype,
                   (hipStream_t)stream, [&](size_t need, int* prc) -> void* {
                       void* w = nullptr;
                       *prc = get_ws(need, ws, ws_bytes, (hipStream_t)stream, &hold, &w);
                       return w;
                   });
}

int tsm2x_split(int64_t m, int64_t k, const float* A, int64_t lda, void* hi, void* lo,
                int64_t ldh, int fmt, void* stream) {
    if (m < 0) return -1;
    if (k < 0) return -2;
    if (!A && m > 0 && k > 0) return -3;
    if (lda < (m > 1 ? m : 1)) return -4;
    if (!hi && m > 0 && k > 0) return -5;
    if (ldh < (m > 1 ? m : 1)) return -7;
    if (fmt != 0 && fmt != 1) return -8;
    if (m == 0 || k == 0) return TSM_SUCCESS;
    launch_split(m, k, A, lda, hi, lo, ldh, fmt, (hipStream_t)stream);
    return check_launch("split_kernel");
}

int tsm2l_split(int transB, int64_t m, int64_t k, int64_t n, const float* A, int64_t lda,
                const float* B, int64_t ldb, float* C, int64_t ldc, void* hi, void* lo,
                int64_t ldh, int fmt, void* stream) {
    if (transB != 0 && transB != 1) return -1;
    if (m < 0) return -2;
    if (k < 0) return -3;
    if (n < 0) return -4;
    if (!A && m > 0 && k > 0) return -5;
    if (lda < (m > 1 ? m : 1)) return -6;
    if (!B && k > 0 && n > 0) return -7;
    if (ldb < ((transB ? n : k) > 1 ? (transB ? n : k) : 1)) return -8;
    if (!C && m > 0 && n > 0) return -9;
    if (ldc < (m > 1 ? m : 1)) return -10;
    if (!hi && m > 0 && k > 0) return -11;
    if (ldh < (m > 1 ? m : 1)) return -13;
    if (fmt != 0 && fmt != 1) return -14;
    if (k > 32 || n > 32 || ((uintptr_t)hi & 7u) || ((uintptr_t)lo & 7u) || ldh % 4)
        return TSM_ERR_UNSUPPORTED;
    if (m == 0) return TSM_SUCCESS;
    hipStream_t st = (hipStream_t)stream;
    if (n == 0 || k == 0) {
        if (n > 0) launch_fill_scale(m, n, C, ldc, 0.0, TSM_F32, st);
        if (k > 0) launch_split(m, k, A, lda, hi, lo, ldh, fmt, st);
        return check_launch("split_kernel");
    }
    LaunchLS L{};
    L.m = m; L.k = (int)k; L.n = (int)n; L.A = A; L.lda = lda; L.hi = (uint16_t*)hi;
    L.lo = (uint16_t*)lo; L.ldh = ldh; L.B = B; L.bsj = transB ? ldb : 1; L.bsp = transB ? 1 : ldb;
    L.C = C; L.ldc = ldc;
    launch_tsm2l_split(L, fmt, st);
    return check_launch("tsm2l_split_kernel");
}

int tsm_kmeans_assign(int64_t m, int64_t k, int64_t n, const void* X, int64_t ldx,
                      int x_rowmajor, const void* Mu, int64_t ldm, int32_t* labels, void* dist,
                      int dtype, void* ws, size_t ws_bytes, void* stream) {
    if (m < 0) return -1;
    if (k < 1 || k > INT32_MAX) return -2;
    if (n < 1 || n > INT32_MAX) return -3;
    if (!X && m > 0) return -4;
    if (x_rowmajor != 0 && x_rowmajor != 1) return -6;
    if (ldx < (x_rowmajor ? k : (m > 1 ? m : 1))) return -5;
    if (!Mu) return -7;
    if (ldm < k) return -8;
    if (!labels && m > 0) return -9;
    if (!plain_dtype(dtype)) return -11;
    if (m == 0) return TSM_SUCCESS;
    void* w = nullptr;
    WsHold hold;
    int rc = get_ws(align256((size_t)n * esize(dtype)), ws, ws_bytes, (hipStream_t)stream, &hold, &w);
    if (rc) return rc;
    LaunchKM L{};
    L.m = m; L.k = k; L.n = n; L.X = X; L.ldx = ldx; L.x_rowmajor = x_rowmajor; L.Mu = Mu;
    L.ldm = ldm; L.mu2 = w;
    L.labels = labels; L.dist = dist; L.cus = cu_count();
    if (launch_kmeans_assign(L, dtype, (hipStream_t)stream)) {
        g_last_hip = "kmeans_assign_kernel: launch failed";
        return TSM_ERR_HIP;
    }
    return TSM_SUCCESS;
}

size_t tsm2x_workspace_size(int op, int64_t m, int64_t k, int64_t n, int dtype) {
    if (op == TSM_OP_KMEANS)
        return (m >= 0 && k >= 1 && n >= 1 && plain_dtype(dtype)) ? align256((size_t)n * esize(dtype)) : 0;
    if (m <= 0 || k <= 0 || n <= 0 || !valid_dtype(dtype)) return 0;
    // products: enough for a B given transposed as well, and for a panel of any
    // width the call may run in (the panels reuse one workspace): a narrower
    // last panel can need more than the others, its split being finer
    auto most = [&](int transA) {
        const bool wide = n > 32 && !transA && plain_dtype(dtype) && m > 32;
        size_t w = 0;
        for (const int64_t p : {n < 32 ? n : (int64_t)32, n > 32 ? n % 32 : (int64_t)0,
                                !wide ? (int64_t)0 : n < 64 ? n : (int64_t)64,
                                wide && n > 64 ? n % 64 : (int64_t)0}) {
            const size_t b = p > 0 ? tsm2r_ws_max(transA, m, k, p, dtype, true) : 0;
            if (b > w) w = b;
        }
        return w;
    };
    switch (op) {
        case TSM_OP_TSM2R: return most(0);
        case TSM_OP_TSM2R_ROWMAJOR: return plain_dtype(dtype) ? most(1) : 0;
        case TSM_OP_TSM2L: return k <= 32 ? 0 : most(0);
        case TSM_OP_GRAD_B: return n <= 32 ? plan_tn(m, k, n, dtype, cu_count()).ws : 0;
        default: return 0;
    }
}

const char* tsm2x_kernel_name(int op, int64_t m, int64_t k, int64_t n, int dtype) {
    if (op != TSM_OP_TSM2R || m <= 0 || k <= 0 || n <= 0 || n > 32 || !plain_dtype(dtype))
        return nullptr;
    if (tt_shape(0, m, k, n, dtype)) return tt_name((int)m, (int)n, dtype);
    NNPlan P{};
    return plan_nn(m, k, n, dtype, cu_count(), true, &P) ? nullptr : P.name;
}

int tsm2x_tsm2r_plan(int64_t m, int64_t k, int64_t n, int dtype, int* slices, int* tall,
                     int64_t* tiles, int* tile_rows, int* occupancy, int* cus) {
    if (m <= 0) return -1;
    if (k <= 0) return -2;
    if (n <= 0 || n > 32) return -3;
    if (!plain_dtype(dtype)) return -4;
    const int c = cu_count();
    NNPlan P{};
    if (plan_nn(m, k, n, dtype, c, true, &P)) return TSM_ERR_UNSUPPORTED;
    if (slices) *slices = P.S;
    if (tall) *tall = P.tall;
    if (tiles) *tiles = P.tiles;
    if (tile_rows) *tile_rows = P.tile_rows;
    if (occupancy) *occupancy = P.occ;
    if (cus) *cus = c;
    return TSM_SUCCESS;
}

int tsm2x_tsm2r_pin(int64_t m, int64_t k, int64_t n, int dtype, int slices, int tall) {
    if (m <= 0) return -1;
    if (k <= 0) return -2;
    if (n <= 0 || n > 32) return -3;
    if (!plain_dtype(dtype)) return -4;
    if (slices < 0 || slices > k) return -5;
    if (tall < -1 || tall > 1) return -6;
    std::lock_guard<std::mutex> lk(g_pin_mu);
    if (slices == 0 && tall == -1)
        g_pins.erase(PinKey(m, k, n, dtype));
    else
        g_pins[PinKey(m, k, n, dtype)] = NNPin{slices, tall};
    return TSM_SUCCESS;
}

const char* tsm2x_error_string(int code) {
    if (code < 0) return "invalid argument (the code is minus its 1-based position)";
    switch (code) {
        case TSM_SUCCESS: return "success";
        case TSM_ERR_UNSUPPORTED: return "shape or storage type outside the supported range";
        case TSM_ERR_HIP: return "a HIP runtime call failed (see tsm2x_last_hip_error)";
        case TSM_ERR_WORKSPACE: return "workspace too small or not 256-byte aligned";
        case TSM_ERR_ALLOC: return "could not allocate the library workspace";
        default: return "unknown error code";
    }
}

const char* tsm2x_last_hip_error(void) { return g_last_hip.c_str(); }

int tsm2x_version(void) { return 100; }

void tsm2x_finalize(void) {
    int cur = 0;
    (void)hipGetDevice(&cur);
    for (size_t d = 0;; ++d) {
        std::map<WsKey, std::shared_ptr<WsBuf>> bufs;
        std::vector<void*> retired;
        {
            std::lock_guard<std::mutex> lk(g_mu);
            if (d >= g_dev.size()) break;
            bufs.swap(g_dev[d].bufs);
            retired.swap(g_dev[d].retired);
        }
        if (bufs.empty() && retired.empty()) continue;
        (void)hipSetDevice((int)d);
        for (auto& e : bufs) {
            std::lock_guard<std::mutex> lk(e.second->mu);
            e.second->dead = true;
            if (e.second->p) (void)hipFree(e.second->p);
            e.second->p = nullptr;
        }
        for (void* p : retired) (void)hipFree(p);
    }
    (void)hipSetDevice(cur);
}

}  // extern "C"

// Host side of libenec: argument checks, kernel dispatch, the parameter search.
// See include/enec.h for the contract of every entry point.
#include "enec.h"
#include "enec_kernels.hpp"

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <tuple>
#include <vector>

namespace enec {

// kernels that exist once: the header-only stream of an empty tensor, zero fill, plain copy
__global__ void compress_empty_kernel(uint8_t *out, uint64_t *out_bytes, uint32_t B, uint32_t b, uint32_t n, uint32_t m,
                                      uint32_t dtype, uint32_t L)
{
    if (threadIdx.x != 0) return;
    uint32_t *h = reinterpret_cast<uint32_t *>(out);
    h[0] = 0x43454E45u;
    h[1] = 1u | (dtype << 16) | ((L & 0xFFu) << 24);
    h[2] = h[3] = 0;
    h[4] = B; h[5] = 0;
    h[6] = b | (n << 8) | (m << 16) | (exponent_bits((int)dtype) << 24);
    h[7] = 0;
    h[8] = 80; h[9] = 0;
    h[10] = L >> 8;                           // 1 = a stream with one tuple per data block
    for (int i = 11; i < 16; ++i) h[i] = 0;
    h[16] = h[17] = h[18] = h[19] = 0;      // table[0] = 0 and the pad to 80 bytes
    if (out_bytes) *out_bytes = 80;
}

__global__ void __launch_bounds__(256) fill_zero_kernel(uint4 *p, uint64_t nvec)
{
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    for (uint64_t v = (uint64_t)blockIdx.x * 256u + threadIdx.x; v < nvec; v += stride)
        p[v] = make_uint4(0, 0, 0, 0);
}

__global__ void __launch_bounds__(256) copy_kernel(uint4 *__restrict__ dst, const uint4 *__restrict__ src, uint64_t nvec)
{
    const uint64_t stride = (uint64_t)gridDim.x * 256u;
    for (uint64_t v = (uint64_t)blockIdx.x * 256u + threadIdx.x; v < nvec; v += stride) dst[v] = src[v];
}

// for a workspace that is not in the state the last call left it in: the tuner's counts, one workgroup per histogram, and the
// number of workgroups that have added theirs
__global__ void __launch_bounds__(128) clear_counts_kernel(uint4 *hist, uint32_t *done)
{
    hist[blockIdx.x * 128u + threadIdx.x] = make_uint4(0, 0, 0, 0);
    if (blockIdx.x == 0 && threadIdx.x == 0) *done = 0;
}

}  // namespace enec

namespace {

using namespace enec;

// workspace: [0, 1024) control records of the block classes | [1024, 33792) sixteen histograms |
// group words | block words (the last two sized by the call's block count)
// (the counting kernel's own counter lies in the last control record, whose first six words only are used otherwise)
constexpr size_t WS_CTL = 0, WS_HIST_DONE = 1008, WS_HIST = 1024, WS_HIST_SLOTS = MAX_BATCH, WS_STATE = WS_HIST + WS_HIST_SLOTS * 256 * 8;
inline size_t ws_groups(size_t nb) { return (nb + GROUP - 1) / GROUP; }
// The state words behind WS_STATE: first the group accumulators, which every call leaves zero, in
// a region whose length depends only on the size of the workspace (1/9 of the words), then the
// tagged group and block words, handed out anew by every launch.
inline size_t ws_state_words(size_t workspace_bytes) { return workspace_bytes < WS_STATE ? 0 : (workspace_bytes - WS_STATE) / 8; }
inline size_t ws_acc_words(size_t workspace_bytes) { return ws_state_words(workspace_bytes) / 9; }
constexpr size_t MAX_ELEMS = (size_t)1 << 34;      // keeps every offset below 2^36 bytes

inline size_t align16(size_t v) { return (v + 15) & ~(size_t)15; }
inline bool block_ok(uint32_t B) { return B >= 2048 && B <= 32768 && (B & (B - 1)) == 0; }
inline uint32_t ilog2(uint32_t v) { uint32_t r = 0; while ((1u << r) < v) ++r; return r; }
inline size_t num_blocks(size_t n, uint32_t B) { return (n + B - 1) / B; }
inline bool dtype_ok(int dtype) { return dtype == ENEC_BF16 || dtype == ENEC_FP16 || dtype == ENEC_FP32; }
inline unsigned exp_bits(int dtype) { return dtype == ENEC_FP16 ? 5u : 8u; }
inline size_t elem_bytes(int dtype) { return dtype == ENEC_FP32 ? 4 : 2; }
// end of header + offset table; an fp32 stream keeps the lower halves of its elements from here on
inline size_t table_end(size_t n, uint32_t B) { return align16(ENEC_HEADER_BYTES + 8 * (num_blocks(n, B) + 1)); }
inline size_t payload_base(size_t n, uint32_t B, int dtype)
{
    return table_end(n, B) + (dtype == ENEC_FP32 ? align16(2 * n) : 0);
}
inline bool aligned16(const void *p) { return ((uintptr_t)p & 15) == 0; }
// a stream with one tuple per data block keeps them (4 bytes each) right behind the offset table
inline size_t tuple_table_bytes(size_t n, uint32_t B) { return align16(4 * num_blocks(n, B)); }

inline bool group_ok(unsigned L) { return L == 8 || L == 16 || L == 32; }

inline CompressFn pick_compress(int m, int a, int dtype, unsigned L, uint32_t B)
{
    const bool std_block = B == 1u << DEFAULT_LOGB;
#define ENEC_PICK(dt, lpg) (std_block ? pick_compress_##dt##_##lpg##_b14(m, a) : pick_compress_##dt##_##lpg##_b0(m, a))
#define ENEC_ROW(dt) (L == 8 ? ENEC_PICK(dt, lpg1) : L == 16 ? ENEC_PICK(dt, lpg2) : ENEC_PICK(dt, lpg4))
    if (dtype == ENEC_FP16) return ENEC_ROW(dt1);
    if (dtype == ENEC_FP32) return ENEC_ROW(dt2);
    return ENEC_ROW(dt0);
#undef ENEC_ROW
#undef ENEC_PICK
}
// A group length needs whole 16-byte vectors of mask per block (B >= 128 L) and at most 64 mask
// words per block (the kernels scan them with one wave: B / L <= 2048).
inline bool group_fits_block(unsigned L, uint32_t B) { return B >= 128u * L && B / L <= 2048u; }

// how the kernels subtract exponents in byte lanes: 0 = plain subtract (no byte can borrow for
// an exponent inside the window), 1 = borrow-safe subtract, the window is the whole exponent
// range, 2 = borrow-safe subtract plus an explicit window test (the window of an 8-bit exponent
// touches 0 or 255, where a plain subtract could wrap back into the window)
inline unsigned subtract_mode(unsigned b, unsigned n, int dtype)
{
    if (n == exp_bits(dtype)) return 1u;
    if (dtype == ENEC_FP16) return 0u;           // 5-bit exponents in byte lanes cannot wrap
    const unsigned cc = b + (1u << (n - 1));
    return (cc <= 255 && cc >= (1u << n) - 1u) ? 0u : 2u;
}

bool device_accessible(const void *p)
{
    hipPointerAttribute_t attr;
    if (hipPointerGetAttributes(&attr, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return attr.type == hipMemoryTypeDevice || attr.type == hipMemoryTypeHost ||
           attr.type == hipMemoryTypeManaged;
}

// Number of workgroups of `fn` the current device holds at once.  The figure depends only on the
// kernel, its launch shape and the device, so it is looked up once per such combination and kept (a
// map under a mutex: there are several hundred kernel instances); a call whose combination is known
// makes no HIP call here, which also keeps it usable under stream capture once warmed up.
unsigned resident_workgroups(const void *fn, unsigned threads, size_t lds)
{
    static std::map<std::tuple<const void *, unsigned, size_t, int>, unsigned> cache;
    static std::mutex mu;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    std::lock_guard<std::mutex> lock(mu);
    const auto key = std::make_tuple(fn, threads, lds, dev);
    const auto hit = cache.find(key);
    if (hit != cache.end()) return hit->second;
    if (lds > 65536 &&
        hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return 0;
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, (int)threads, lds) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || per_cu < 1 || cus < 1)
        return 0;
    const unsigned value = (unsigned)per_cu * (unsigned)cus;
    cache.emplace(key, value);
    return value;
}

// The persistent grid of a compression launch for `total` blocks on a device that holds `resident` workgroups.
// (Shrinking the grid until every round of blocks is full, e.g. 727 instead of 768 workgroups for 12352 blocks, was
// measured and lost 1.5 % on the 7B layer: the last, nearly empty round costs less than the parallelism given up
// in all the others.)
unsigned persistent_grid(unsigned total, unsigned resident)
{
    return total < resident ? total : resident;
}

// polls after which a waiting workgroup gives up; builds with ENEC_TEST_HOOKS (the test library) let
// the environment lower it so that a test can watch a scan give up without waiting for seconds
uint32_t spin_limit()
{
#ifdef ENEC_TEST_HOOKS
    if (const char *e = std::getenv("ENEC_SPIN_LIMIT")) {
        const long v = std::atol(e);
        if (v > 0 && v < (long)SPIN_LIMIT) return (uint32_t)v;
    }
#endif
    return SPIN_LIMIT;
}

// The next item of a launch of a kernel with deferred stores; a.B is set.  acc / word: the first accumulator and scan word
// that are still free (tags make their reuse from one launch to the next safe).
void fill_compress_item(CompressArgs &a, size_t &acc, size_t &word, void *workspace, const void *in, void *out, uint64_t *out_bytes,
                        size_t n_elems, int dtype)
{
    CompressItem &c = a.item[a.n_items++];
    uint64_t *state = reinterpret_cast<uint64_t *>(static_cast<uint8_t *>(workspace) + WS_STATE);
    c.nb = (uint32_t)num_blocks(n_elems, a.B);
    c.in = static_cast<const uint16_t *>(in);
    c.out = static_cast<uint8_t *>(out);
    c.out_bytes = out_bytes;
    c.ws_acc = state + acc;
    acc += ws_groups(c.nb);
    c.ws_group = state + word;
    word += ws_groups(c.nb);
    c.ws_block = state + word;
    word += c.nb;
    c.n_elems = n_elems;
    c.payload_base = payload_base(n_elems, a.B, dtype);
    c.tail_base = table_end(n_elems, a.B);
    c.first = a.total;
    a.total += c.nb;
}

template <class Fn>
void launch_compress(Fn fn, CompressArgs &a, unsigned resident, unsigned threads, size_t lds, hipStream_t s)
{
    // (tensors of one block come on top of the grid, which may leave workgroups waiting until one of theirs ends: these draw
    // their first block then)
    const unsigned grid = persistent_grid(a.total, resident);
    a.wgs = grid;
    a.ncls = grid < 8 ? grid : 8;
    // The next ticket is drawn while the current block is worked on only if there are blocks for
    // two rounds: with fewer, an early workgroup would take the block of one that starts a moment later.
    a.lookahead = a.total >= 2 * grid ? 1u : 0u;
    a.spin_limit = spin_limit();
    hipLaunchKernelGGL(fn, dim3(grid + a.n_single), dim3(threads), lds, s, a);
}

// Dynamic LDS of a decompression workgroup of a 16-bit format, so that a CU works on 65536 elements at a time (the
// reason is in enec_decompress.hpp): too much for one workgroup more, little enough for these.  Blocks of 2048
// elements need none, the CU's 32 waves are their limit.
constexpr size_t LDS_PER_CU = 160 * 1024, LDS_UNIT = 1280;     // bytes, and the step in which they are handed out
constexpr size_t decompress_lds_floor(uint32_t B) { return B <= 2048 ? 0 : LDS_PER_CU / (65536 / B + 1) + 256; }
constexpr bool holds_65536_elements(uint32_t B)
{
    const size_t each = (decompress_lds_floor(B) + LDS_UNIT - 1) / LDS_UNIT * LDS_UNIT;
    return LDS_PER_CU / each == 65536 / B && each <= 65536;    // (more than 64 KB would have to be asked for)
}
static_assert(holds_65536_elements(4096) && holds_65536_elements(8192) && holds_65536_elements(16384) &&
                  holds_65536_elements(32768), "LDS of a decompression workgroup");

// Pinned memory in which a call that tunes finds its counts: the counting kernel stores them there, where a copy to pageable
// memory takes 14 us.  A call takes a slot for as long as it runs; up to four are kept for later calls, for
// all threads, streams and devices, more are given back when their call ends, and these when the process does.
class CountSlots {
    // Another thread may be capturing a graph: allocating or freeing would end its capture in any mode but this one.
    struct SparesCaptures {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool swapped = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        ~SparesCaptures() { if (swapped) { hipStreamCaptureMode back = mode; (void)hipThreadExchangeStreamCaptureMode(&back); } }
    };
public:
    // the counts of WS_HIST_SLOTS tensors, then the word that says that they have arrived
    static constexpr size_t ARRIVED = WS_HIST_SLOTS * 256 * 8, BYTES = ARRIVED + 64, KEPT = 4;
    void *take()
    {
        {
            std::lock_guard<std::mutex> lock(mu_);
            if (!free_.empty()) {
                void *p = free_.back();
                free_.pop_back();
                return p;
            }
        }
        const SparesCaptures guard;
        void *p = nullptr;
        if (hipHostMalloc(&p, BYTES, hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) { (void)hipGetLastError(); p = nullptr; }
        return p;
    }
    void give(void *p)
    {
        {
            std::lock_guard<std::mutex> lock(mu_);
            if (free_.size() < KEPT) { free_.push_back(p); return; }
        }
        const SparesCaptures guard;
        if (hipHostFree(p) != hipSuccess) (void)hipGetLastError();        // (nobody's launch failed)
    }
    CountSlots() { free_.reserve(KEPT); }
    ~CountSlots() { for (void *p : free_) (void)hipHostFree(p); }
private:
    std::mutex mu_;
    std::vector<void *> free_;
};
// made by the first call that tunes, after the runtime has started, so that it ends before the runtime does
CountSlots &count_slots() { static CountSlots slots; return slots; }

// elements that the parameter search looks at: those of every `every`-th chunk, the first one included
uint64_t sampled_elements(uint64_t n, uint32_t every)
{
    const uint64_t chunks = (n + SAMPLE_CHUNK - 1) / SAMPLE_CHUNK;
    if (chunks == 0) return 0;
    const uint64_t picked = (chunks + every - 1) / every;
    const bool last = (chunks - 1) % every == 0;             // the last chunk, perhaps a short one, is among them
    return picked * SAMPLE_CHUNK - (last ? chunks * SAMPLE_CHUNK - n : 0);
}

unsigned bit_length(unsigned v) { return v ? 32u - (unsigned)__builtin_clz(v) : 0u; }

// ---- Sec. V-E phases 1-3 on a 256-bin exponent histogram -------------------------------------
struct Search {
    unsigned lo, hi;            // occupied exponent range [l, h] (phase 1)
    uint64_t total;             // number of elements
    unsigned b, n;              // mapping centre and stored width (phase 2)
    unsigned m, L;              // threshold width and group length (phase 3)
    uint64_t at_most[9];        // at_most[w] = elements whose y fits in w bits, w = 0 .. n
};

// Phase 2: every centre b of [l, h] with the width Eq. 1 gives it (capped at the exponent field) is
// priced by Eq. 3 in exact integers, sum of count * y with y from Eq. 2; the cheapest wins, then the
// narrower, then the smaller centre.  Afterwards the elements are counted by the bit length of their y,
// which is all phase 3 needs.  False for an empty histogram.
// With the width fixed, the cost D(b) of the next centre follows from the one before: every y grows by one, and those of
// the values congruent to b + 1 modulo 2^n fall from 2^n - 1 to 0, so D(b + 1) = D(b) + total - 2^n H[(b + 1) mod 2^n] with
// the counts H folded modulo 2^n (unsigned arithmetic, exact).  Two or three widths occur among the centres.
bool centre_and_width(const uint64_t *hist, unsigned nmax, Search &r)
{
    r.lo = 256; r.hi = 0; r.total = 0;
    for (unsigned x = 0; x < 256; ++x) {
        if (!hist[x]) continue;
        if (r.lo == 256) r.lo = x;
        r.hi = x;
        r.total += hist[x];
    }
    if (r.total == 0) return false;
    auto width_of = [&](unsigned b) {
        const unsigned need_below = bit_length(b - r.lo);                       // y = b - x, largest for x = l
        const unsigned need_above = r.hi > b ? bit_length(r.hi - b - 1u) : 0u;  // y = 2^n - (x - b)
        const unsigned n = (need_below > need_above ? need_below : need_above) + 1u;
        return n < nmax ? n : nmax;
    };
    unsigned widths = 0;
    for (unsigned b = r.lo; b <= r.hi; ++b) widths |= 1u << width_of(b);
    auto best = std::make_tuple(~(uint64_t)0, 0u, 0u);
    for (unsigned n = 1; n <= nmax; ++n) {
        if (!(widths >> n & 1u)) continue;
        const unsigned mask = (1u << n) - 1u;
        uint64_t folded[256] = {}, cost = 0;
        for (unsigned x = r.lo; x <= r.hi; ++x) {
            folded[x & mask] += hist[x];
            cost += hist[x] * (uint64_t)((r.lo - x) & mask);
        }
        for (unsigned b = r.lo; b <= r.hi; ++b) {
            if (b != r.lo) cost += r.total - (folded[b & mask] << n);
            if (width_of(b) != n) continue;
            const auto k = std::make_tuple(cost, n, b);
            if (k < best) best = k;               // lexicographic: cost, then width, then centre
        }
    }
    r.n = std::get<1>(best);
    r.b = std::get<2>(best);
    uint64_t by_length[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (unsigned x = r.lo; x <= r.hi; ++x) by_length[bit_length((r.b - x) & ((1u << r.n) - 1u))] += hist[x];
    uint64_t run = 0;
    for (unsigned w = 0; w <= r.n; ++w) { run += by_length[w]; r.at_most[w] = run; }
    return true;
}

// Phase 3, Eq. 4: expected exponent bits per element 1/L + n + (m - n) p(m)^L over m in [0, n] and the
// candidate group lengths (OR of 8, 16, 32), p(m) = share of elements with y < 2^m.  Evaluated in IEEE
// double, p^L by log2 L squarings, as (1/L + n) + (m - n) p^L; the smallest wins, then the smaller m,
// then the smaller L.  (The build keeps the compiler from fusing the multiply and the add.)
void threshold_and_length(Search &r, uint32_t lengths)
{
    bool have = false;
    double least = 0.0;
    for (unsigned L = 8, squarings = 3; L <= 32; L *= 2, ++squarings) {
        if (!(lengths & L)) continue;
        for (unsigned m = 0; m <= r.n; ++m) {
            double q = (double)r.at_most[m] / (double)r.total;
            for (unsigned i = 0; i < squarings; ++i) q = q * q;
            const double bits = (1.0 / (double)L + (double)r.n) + ((double)m - (double)r.n) * q;
            if (!have || bits < least || (bits == least && (m < r.m || (m == r.m && L < r.L)))) {
                have = true; least = bits; r.m = m; r.L = L;
            }
        }
    }
}

// the tuple for a histogram; the number of elements in it
uint64_t search(const uint64_t *hist, int dtype, uint32_t lengths, enec_params *params)
{
    Search r;
    const bool any = centre_and_width(hist, exp_bits(dtype), r);
    if (!any) {                                                 // no elements at all: (b, n) = (0, 1) and p = 1
        r.b = 0; r.n = 1; r.total = 1;
        r.at_most[0] = r.at_most[1] = 1;
    }
    threshold_and_length(r, lengths);
    *params = enec_params{(uint8_t)r.b, (uint8_t)r.n, (uint8_t)r.m, (uint8_t)r.L};
    return any ? r.total : 0;
}

struct Header {
    enec_params prm;
    uint64_t n_elems, total;
    uint32_t B, nb, status;
    int dtype;
    bool per_block;          // one tuple per data block (header byte 40)
};

int parse_header(const void *host_header, Header *h)
{
    const uint8_t *p = static_cast<const uint8_t *>(host_header);
    if (std::memcmp(p, "ENEC", 4) != 0) return ENEC_E_FORMAT;
    uint16_t ver; std::memcpy(&ver, p + 4, 2);
    if (ver != 1 || !group_ok(p[7])) return ENEC_E_FORMAT;
    h->dtype = p[6];
    if (!dtype_ok(h->dtype)) return ENEC_E_DTYPE;
    if (p[27] != exp_bits(h->dtype)) return ENEC_E_FORMAT;
    std::memcpy(&h->n_elems, p + 8, 8);
    std::memcpy(&h->B, p + 16, 4);
    std::memcpy(&h->nb, p + 20, 4);
    h->prm.b = p[24]; h->prm.n = p[25]; h->prm.m = p[26]; h->prm.L = p[7];
    std::memcpy(&h->status, p + 28, 4);
    std::memcpy(&h->total, p + 32, 8);
    if (p[40] > 1) return ENEC_E_FORMAT;
    h->per_block = p[40] == 1;
    return ENEC_OK;
}

}  // namespace

extern "C" {

uint32_t enec_version(void) { return 1; }

const char *enec_strerror(int status)
{
    switch (status) {
    case ENEC_OK: return "ok";
    case ENEC_E_ARG: return "invalid argument (null or misaligned pointer, size out of range)";
    case ENEC_E_DTYPE: return "unsupported dtype (bf16, fp16 and fp32 are supported)";
    case ENEC_E_BLOCK: return "block_size must be a power of two in [2048, 32768]";
    case ENEC_E_PARAMS: return "invalid parameters (need 1 <= n <= exponent width, 0 <= m <= n, b inside the exponent range, L in {8, 16, 32} with 128 L <= block_size <= 2048 L)";
    case ENEC_E_CAPACITY: return "output capacity or workspace too small";
    case ENEC_E_RANGE: return "an exponent lies outside the window of (b, n)";
    case ENEC_E_FORMAT: return "not an ENEC stream or header mismatch";
    case ENEC_E_HIP: return "HIP runtime error (as a stream's status: the inter-block scan gave up on a workspace that was not in the state the last call left it in)";
    default: return "unknown status";
    }
}

uint32_t enec_default_block_size(size_t n_elems)
{
    uint32_t B = ENEC_DEFAULT_BLOCK;
    while (B > 2048 && B > n_elems) B >>= 1;
    return B;
}

size_t enec_compress_bound(size_t n_elems, int dtype, uint32_t block_size)
{
    if (!dtype_ok(dtype)) return 0;
    const uint32_t B = block_size ? block_size : enec_default_block_size(n_elems);
    if (!block_ok(B)) return 0;
    // worst case for any group length: every group anomalous at full exponent width (fp16: (5 + 3)
    // plane bits) and the longest mask (L = 8)
    return payload_base(n_elems, B, dtype) + num_blocks(n_elems, B) * align16((size_t)B + B / 64 + B);
}

size_t enec_workspace_bytes(size_t n_elems, uint32_t block_size)
{
    const uint32_t B = block_size ? block_size : enec_default_block_size(n_elems);
    if (!block_ok(B)) return 0;
    // room for the scan words of up to MAX_BATCH tensors with n_elems elements in total
    const size_t nb = num_blocks(n_elems, B) + MAX_BATCH;
    const size_t groups = ws_groups(nb) + MAX_BATCH;
    const size_t by_acc = 9 * groups, by_words = (9 * (groups + nb) + 7) / 8;
    return (WS_STATE + 8 * ((by_acc > by_words ? by_acc : by_words) + 9) + 255) & ~(size_t)255;
}

int enec_workspace_init(void *workspace, size_t bytes, void *stream)
{
    if (!workspace || !aligned16(workspace) || (bytes & 15)) return ENEC_E_ARG;
    if (bytes == 0) return ENEC_OK;
    const uint64_t nvec = bytes / 16;
    const unsigned grid = (unsigned)((nvec + 255) / 256 < 1024 ? (nvec + 255) / 256 : 1024);
    fill_zero_kernel<<<grid, 256, 0, (hipStream_t)stream>>>(static_cast<uint4 *>(workspace), nvec);
    return hipGetLastError() == hipSuccess ? ENEC_OK : ENEC_E_HIP;
}

int enec_tune_histogram(const uint64_t *hist, int dtype, enec_params *params)
{
    return enec_tune_histogram_groups(hist, dtype, 16u, 0u, params);
}

int enec_tune_histogram_groups(const uint64_t *hist, int dtype, uint32_t group_lengths, uint32_t block_size,
                               enec_params *params)
{
    if (!dtype_ok(dtype)) return ENEC_E_DTYPE;
    if (!hist || !params) return ENEC_E_ARG;
    if (!(group_lengths & (8u | 16u | 32u)) || (group_lengths & ~(8u | 16u | 32u))) return ENEC_E_PARAMS;
    const uint32_t B = block_size ? block_size : ENEC_DEFAULT_BLOCK;
    if (!block_ok(B)) return ENEC_E_BLOCK;
    // only lengths the block size admits are candidates; 16 fits every block size and stands in if none is left
    uint32_t lengths = 0;
    for (unsigned L = 8; L <= 32; L *= 2)
        if ((group_lengths & L) && group_fits_block(L, B)) lengths |= L;
    if (!lengths) lengths = 16u;
    search(hist, dtype, lengths, params);
    return ENEC_OK;
}

int enec_tune_batch(const enec_tune_item *items, size_t n_items, int dtype, uint32_t every, enec_params *params,
                    uint64_t *histograms, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!dtype_ok(dtype)) return ENEC_E_DTYPE;
    if (workspace_bytes < WS_STATE) return ENEC_E_CAPACITY;
    if ((!items && n_items) || (!params && n_items) || !workspace || !aligned16(workspace) || every == 0) return ENEC_E_ARG;
    for (size_t i = 0; i < n_items; ++i)
        if ((!items[i].in && items[i].n_elems) || !aligned16(items[i].in) || items[i].n_elems > MAX_ELEMS) return ENEC_E_ARG;
    hipStream_t s = (hipStream_t)stream;
    auto *dhist = reinterpret_cast<unsigned long long *>(static_cast<uint8_t *>(workspace) + WS_HIST);
    if (n_items == 0) return ENEC_OK;
    // a capture cannot be waited for: refused before anything is enqueued into it
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(s, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
        (void)hipGetLastError();
        return ENEC_E_HIP;
    }
    uint64_t *host = static_cast<uint64_t *>(count_slots().take());
    if (!host) return ENEC_E_HIP;
    // sixteen tensors at a time: their histograms are counted into sixteen slots, handed over together,
    // and the stream is waited for once
    for (size_t first = 0; first < n_items; first += WS_HIST_SLOTS) {
        const size_t count = n_items - first < WS_HIST_SLOTS ? n_items - first : WS_HIST_SLOTS;
        // One launch for the sixteen: a workgroup per HIST_THREADS vectors of the sample, or HIST_WORKGROUPS shared out
        // by size, rounded down but at least one for each tensor (so up to fifteen more).
        HistogramArgs a;
        a.n_items = 0;
        a.every = every;
        uint64_t want_all = 0;
        for (size_t j = 0; j < count; ++j)
            want_all += (items[first + j].n_elems * elem_bytes(dtype) / 16 / every + HIST_THREADS - 1) / HIST_THREADS;
        uint32_t grid = 0;
        for (size_t j = 0; j < count; ++j) {
            const enec_tune_item &it = items[first + j];
            if (it.n_elems == 0) continue;
            const uint64_t want = (it.n_elems * elem_bytes(dtype) / 16 / every + HIST_THREADS - 1) / HIST_THREADS;
            uint64_t share = want_all > HIST_WORKGROUPS ? want * HIST_WORKGROUPS / want_all : want;
            if (share < 1) share = 1;
            HistogramItem &d = a.item[a.n_items++];
            d.in = it.in;
            d.n_elems = it.n_elems;
            d.hist = dhist + 256 * j;
            d.first = grid;
            d.count = (uint32_t)share;
            grid += d.count;
        }
        volatile uint32_t *arrived = reinterpret_cast<volatile uint32_t *>(host + CountSlots::ARRIVED / 8);
        *arrived = 0;
        if (grid) {
            for (uint32_t j = a.n_items; j < (uint32_t)MAX_BATCH; ++j) a.item[j] = a.item[0];
            a.done = reinterpret_cast<uint32_t *>(static_cast<uint8_t *>(workspace) + WS_HIST_DONE);
            a.counts = dhist;
            a.host = reinterpret_cast<unsigned long long *>(host);
            a.arrived = const_cast<uint32_t *>(arrived);
            a.n_counts = (uint32_t)count * 256u;
            a.wgs = grid;
        } else {
            std::memset(host, 0, count * 256 * 8);
        }
        const void *fn = dtype == ENEC_FP32 ? (const void *)histogram_kernel<DT_FP32>
                       : dtype == ENEC_FP16 ? (const void *)histogram_kernel<DT_FP16> : (const void *)histogram_kernel<DT_BF16>;
        // Every call leaves the counters zero.  A workspace in which they were not would show in the sums, or in a kernel that
        // ends without handing over: it is cleared then, and counted once more.  Counts that are wrong even so (something writes
        // to the workspace during the call) are not used.
        // (Looking for `arrived` instead of waiting for the stream takes 5 us less for the layer, and the runtime makes up for 2
        // of them in whatever is called next; hipStreamQuery or the wait after the search take more than the wait here.)
        bool sound = false;
        enec_params found[WS_HIST_SLOTS];
        for (int attempt = 0; attempt < 2 && !sound; ++attempt) {
            bool launched = true;
            if (attempt) {
                *arrived = 0;
                uint4 *counts = reinterpret_cast<uint4 *>(dhist);
                void *args[] = {&counts, &a.done};
                launched = hipLaunchKernel((const void *)clear_counts_kernel, dim3((unsigned)count), dim3(128), args, 0, s) == hipSuccess;
            }
            void *args[] = {&a};
            if (launched && grid) launched = hipLaunchKernel(fn, dim3(grid), dim3(HIST_THREADS), args, 0, s) == hipSuccess;
            if (!launched) {                   // (nothing that is still to run writes to the slot)
                (void)hipGetLastError();
                count_slots().give(host);
                return ENEC_E_HIP;
            }
            if (hipStreamSynchronize(s) != hipSuccess) {
                (void)hipGetLastError();
                return ENEC_E_HIP;             // (the slot is not given back: a kernel may still be about to write there)
            }
            sound = !grid || *arrived;
            for (size_t j = 0; j < count && sound; ++j)
                sound = search(host + 256 * j, dtype, 16u, &found[j]) == sampled_elements(items[first + j].n_elems, every);
        }
        if (!sound) {
            count_slots().give(host);
            return ENEC_E_HIP;
        }
        std::copy(found, found + count, params + first);
        if (histograms) std::memcpy(histograms + 256 * first, host, count * 256 * 8);
    }
    count_slots().give(host);
    return ENEC_OK;
}

int enec_tune_sampled(const void *in, size_t n_elems, int dtype, uint32_t every, enec_params *params,
                      uint64_t *histogram, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!params) return ENEC_E_ARG;
    enec_tune_item it;
    it.in = in;
    it.n_elems = n_elems;
    return enec_tune_batch(&it, 1, dtype, every, params, histogram, workspace, workspace_bytes, stream);
}

int enec_tune(const void *in, size_t n_elems, int dtype, enec_params *params, uint64_t *histogram,
              void *workspace, size_t workspace_bytes, void *stream)
{
    return enec_tune_sampled(in, n_elems, dtype, 1, params, histogram, workspace, workspace_bytes, stream);
}

int enec_compress_sampled(const void *in, size_t n_elems, int dtype, uint32_t block_size, uint32_t every,
                          enec_params *params_used, void *out, size_t out_capacity, void *workspace,
                          size_t workspace_bytes, void *stream)
{
    enec_params prm;
    int rc = enec_tune_sampled(in, n_elems, dtype, every, &prm, nullptr, workspace, workspace_bytes, stream);
    if (rc != ENEC_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    for (int attempt = 0; attempt < 2; ++attempt) {
        rc = enec_compress(in, n_elems, dtype, block_size, &prm, out, out_capacity, nullptr, workspace,
                           workspace_bytes, stream);
        if (rc != ENEC_OK) return rc;
        uint8_t head[ENEC_HEADER_BYTES];
        if (hipMemcpyAsync(head, out, sizeof head, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return ENEC_E_HIP;
        uint32_t status = 0;
        rc = enec_stream_info(head, nullptr, nullptr, nullptr, nullptr, nullptr, &status);
        if (rc != ENEC_OK) return rc;
        if (params_used) *params_used = prm;
        if (status != (uint32_t)ENEC_E_RANGE) return (int)status;
        // an exponent outside the sample's window: the full width makes the map a bijection [Sec. V-C]
        prm.n = (uint8_t)exp_bits(dtype);
    }
    return ENEC_E_RANGE;   // not reached: the full width has no range error
}

int enec_compress_batch(const enec_compress_item *items, size_t n_items, int dtype, void *workspace,
                        size_t workspace_bytes, void *stream)
{
    hipStream_t s = (hipStream_t)stream;
    if (!dtype_ok(dtype)) return ENEC_E_DTYPE;
    if (!items || !workspace || !aligned16(workspace)) return ENEC_E_ARG;

    // ---- every check that can be made on the host, before anything is enqueued -------------
    struct Prepared { enec_params prm; uint32_t B; uint32_t nb; };
    std::vector<Prepared> prep(n_items);
    size_t state_words = 0, groups = 0;
    for (size_t i = 0; i < n_items; ++i) {
        const enec_compress_item &it = items[i];
        if (!it.out || (!it.in && it.n_elems) || !aligned16(it.in) || !aligned16(it.out) ||
            it.n_elems > MAX_ELEMS || ((uintptr_t)it.out_bytes & 7))
            return ENEC_E_ARG;
        const uint32_t B = it.block_size ? it.block_size : enec_default_block_size(it.n_elems);
        if (!block_ok(B)) return ENEC_E_BLOCK;
        prep[i].B = B;
        prep[i].nb = (uint32_t)num_blocks(it.n_elems, B);
        state_words += ws_groups(prep[i].nb) + prep[i].nb;
        groups += ws_groups(prep[i].nb);
    }
    const size_t acc_words = ws_acc_words(workspace_bytes);
    if (groups > acc_words || acc_words + state_words > ws_state_words(workspace_bytes)) return ENEC_E_CAPACITY;
    {   // tensors without a tuple are tuned first, together (one wait for the stream per sixteen of them)
        std::vector<enec_tune_item> todo;
        std::vector<size_t> who;
        for (size_t i = 0; i < n_items; ++i)
            if (!items[i].params) {
                enec_tune_item t;
                t.in = items[i].in;
                t.n_elems = items[i].n_elems;
                todo.push_back(t);
                who.push_back(i);
            }
        if (!todo.empty()) {
            std::vector<enec_params> found(todo.size());
            int rc = enec_tune_batch(todo.data(), todo.size(), dtype, 1, found.data(), nullptr, workspace, workspace_bytes, s);
            if (rc != ENEC_OK) return rc;
            for (size_t j = 0; j < who.size(); ++j) prep[who[j]].prm = found[j];
        }
    }
    for (size_t i = 0; i < n_items; ++i) {
        const enec_compress_item &it = items[i];
        if (it.params) prep[i].prm = *it.params;
        const enec_params &prm = prep[i].prm;
        if (prm.n < 1 || prm.n > exp_bits(dtype) || prm.m > prm.n || prm.b >= (1u << exp_bits(dtype)) ||
            !group_ok(prm.L) || !group_fits_block(prm.L, prep[i].B))
            return ENEC_E_PARAMS;
        if (it.out_capacity < enec_compress_bound(it.n_elems, dtype, prep[i].B)) return ENEC_E_CAPACITY;
        if (it.out_bytes && !device_accessible(it.out_bytes)) return ENEC_E_ARG;
    }

    // ---- one launch per group of tensors that share (m, n - m, L, block size) ----------------
    // A tensor of one block whose (m, n - m, L, block size) no longer tensor has is coded without the machinery for the order
    // of blocks (compress_one_block, whatever its tuple and block size): by the first workgroups of the first launch of the same L
    // whose kernel takes such tensors along (takes_singles), has room for it among its arguments and LDS for its records, or,
    // where there is none, with others of its kind in a launch of their own, after the others.  Its own launch behind that of a
    // layer of 405 MB took 4 us for two norm vectors (139.6 -> 135.4 us with the kernel's own gain).
    auto kernel_of = [&](size_t j) {
        return prep[j].B << 16 | (uint32_t)prep[j].prm.n << 12 | (uint32_t)prep[j].prm.m << 8 | prep[j].prm.L;
    };
    std::vector<uint32_t> large;                 // the kernels that tensors of several blocks need
    for (size_t i = 0; i < n_items; ++i)
        if (prep[i].nb > 1 && std::find(large.begin(), large.end(), kernel_of(i)) == large.end()) large.push_back(kernel_of(i));
    auto alone = [&](size_t j) { return prep[j].nb == 1 && std::find(large.begin(), large.end(), kernel_of(j)) == large.end(); };
    std::vector<char> done(n_items, 0);
    auto take_single = [&](SingleItem &c, size_t j) {
        const enec_params &prm = prep[j].prm;
        c.in = static_cast<const uint16_t *>(items[j].in);
        c.out = static_cast<uint8_t *>(items[j].out);
        c.out_bytes = items[j].out_bytes;
        c.n_elems = items[j].n_elems;
        c.payload_base = (uint32_t)payload_base(items[j].n_elems, prep[j].B, dtype);
        c.tail_base = (uint32_t)table_end(items[j].n_elems, prep[j].B);
        c.logB = ilog2(prep[j].B);
        c.b = prm.b; c.n = prm.n; c.m = prm.m;
        c.mode = subtract_mode(prm.b, prm.n, dtype);
        done[j] = 1;
        return (size_t)single_lds_bytes(prep[j].B, prm.L, prm.n - prm.m);
    };
    for (size_t i = 0; i < n_items; ++i) {
        if (done[i] || alone(i)) continue;
        if (prep[i].nb == 0) {
            compress_empty_kernel<<<1, 64, 0, s>>>(static_cast<uint8_t *>(items[i].out), items[i].out_bytes,
                                                   prep[i].B, prep[i].prm.b, prep[i].prm.n, prep[i].prm.m,
                                                   (uint32_t)dtype, prep[i].prm.L);
            done[i] = 1;
            continue;
        }
        CompressArgs a{};
        a.ws_ctl = reinterpret_cast<uint32_t *>(static_cast<uint8_t *>(workspace) + WS_CTL);
        a.B = prep[i].B;
        a.logB = ilog2(a.B);
        size_t word = acc_words, acc = 0;   // scan words handed out to this launch (tags make reuse between launches safe)
        for (size_t j = i; j < n_items && a.n_items < (uint32_t)MAX_BATCH; ++j) {
            if (done[j] || prep[j].nb == 0 || kernel_of(j) != kernel_of(i)) continue;
            fill_compress_item(a, acc, word, workspace, items[j].in, items[j].out, items[j].out_bytes, items[j].n_elems, dtype);
            CompressItem &c = a.item[a.n_items - 1];
            c.b = prep[j].prm.b;
            c.mode = subtract_mode(prep[j].prm.b, prep[j].prm.n, dtype);
            done[j] = 1;
        }
        CompressFn fn = pick_compress(prep[i].prm.m, prep[i].prm.n - prep[i].prm.m, dtype, prep[i].prm.L, a.B);
        if (!fn) return ENEC_E_PARAMS;
        const unsigned threads = a.B / 64 < 64 ? 64 : a.B / 64;
        const size_t plane_bits = prep[i].prm.n + (dtype == ENEC_FP16 ? 3 : 0);
        // two images of the packed part, and the sign/mantissa bytes of the block that waits to be stored
        const size_t lds = 2 * ((size_t)a.B / (8 * prep[i].prm.L) + plane_bits * a.B / 8) +
                           (compress_sm_in_lds(dtype, a.B == 1u << DEFAULT_LOGB) ? a.B : 0);
        const unsigned resident = resident_workgroups((const void *)fn, threads, lds);
        if (resident == 0) return ENEC_E_HIP;
        if (takes_singles(prep[i].prm.m, prep[i].prm.n - prep[i].prm.m, a.logB))
            for (size_t j = 0; j < n_items && a.takes_another_single(); ++j)
                if (!done[j] && alone(j) && prep[j].prm.L == prep[i].prm.L &&
                    single_lds_bytes(prep[j].B, prep[j].prm.L, prep[j].prm.n - prep[j].prm.m) <= lds)
                    take_single(a.single(a.n_single++), j);
        launch_compress(fn, a, resident, threads, lds, s);
    }
    for (size_t i = 0; i < n_items; ++i) {
        if (done[i]) continue;
        SingleArgs sa;
        size_t count = 0, lds = 0;
        uint32_t largest = 0;
        for (size_t j = i; j < n_items && count < (size_t)MAX_BATCH; ++j) {
            if (done[j] || prep[j].prm.L != prep[i].prm.L) continue;
            lds = std::max(lds, take_single(sa.item[count++], j));
            largest = std::max(largest, prep[j].B);
        }
        const SingleFn fn = pick_compress_single(dtype, prep[i].prm.L);
        const SingleFewFn few = pick_compress_single_few(dtype, prep[i].prm.L);
        if (!fn || !few) return ENEC_E_PARAMS;
        const unsigned threads = std::min(largest / 8, SINGLE_THREADS);
        // (a block of 32768 elements whose records hold whole exponents: more than 64 KB has to be asked for)
        const bool is_few = count <= (size_t)SINGLE_FEW;
        if (lds > 65536 && resident_workgroups(is_few ? (const void *)few : (const void *)fn, threads, lds) == 0) return ENEC_E_HIP;
        for (size_t j = count; j < (size_t)(is_few ? SINGLE_FEW : MAX_BATCH); ++j) sa.item[j] = SingleItem{};
        if (is_few) {
            SingleFewArgs fa;
            std::copy_n(sa.item, SINGLE_FEW, fa.item);
            hipLaunchKernelGGL(few, dim3((unsigned)count), dim3(threads), lds, s, fa);
        } else {
            hipLaunchKernelGGL(fn, dim3((unsigned)count), dim3(threads), lds, s, sa);
        }
    }
    return hipGetLastError() == hipSuccess ? ENEC_OK : ENEC_E_HIP;
}

int enec_compress(const void *in, size_t n_elems, int dtype, uint32_t block_size,
                  const enec_params *params, void *out, size_t out_capacity, uint64_t *out_bytes,
                  void *workspace, size_t workspace_bytes, void *stream)
{
    enec_compress_item it;
    it.in = in; it.n_elems = n_elems; it.block_size = block_size; it.params = params;
    it.out = out; it.out_capacity = out_capacity; it.out_bytes = out_bytes;
    return enec_compress_batch(&it, 1, dtype, workspace, workspace_bytes, stream);
}

// ---- enec_compress for callers that cannot allocate: the workspace is the library's own array ----
}  // extern "C"

namespace {

// Scan state, ticket counters and call tags of enec_compress_static: one array per GPU, held until the
// process ends.  In host code the array's name stands for the symbol, not for device memory; the
// address on a device comes from hipGetSymbolAddress with that device current, once per device.
static __device__ __align__(256) uint8_t scratch[ENEC_STATIC_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
void *scratch_ptr[MAX_DEVICES];       // per device: the array's address there, null until its first call
std::mutex scratch_mu;

// address of `scratch` on the current device; the first call on a device looks it up and enqueues
// the fill kernel that brings the array into the state enec_workspace_init leaves a workspace in
int static_scratch(hipStream_t s, void **out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) { (void)hipGetLastError(); return ENEC_E_HIP; }
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) { (void)hipGetLastError(); return ENEC_E_HIP; }
        const int rc = enec_workspace_init(ptr, ENEC_STATIC_SCRATCH_BYTES, s);
        if (rc != ENEC_OK) return rc;
        scratch_ptr[dev] = ptr;
    }
    *out = scratch_ptr[dev];
    return ENEC_OK;
}

}  // namespace

extern "C" {

int enec_compress_static(const void *in, size_t n_elems, int dtype, uint32_t block_size, const enec_params *params,
                         void *out, size_t out_capacity, uint64_t *out_bytes, void *stream)
{
    if (!params) return ENEC_E_ARG;                       // tuning waits for the stream: not for these callers
    if (!dtype_ok(dtype)) return ENEC_E_DTYPE;
    const uint32_t B = block_size ? block_size : enec_default_block_size(n_elems);
    if (!block_ok(B)) return ENEC_E_BLOCK;
    if (n_elems > MAX_ELEMS) return ENEC_E_ARG;
    if (enec_workspace_bytes(n_elems, B) > ENEC_STATIC_SCRATCH_BYTES) return ENEC_E_CAPACITY;
    void *ws = nullptr;
    const int rc = static_scratch((hipStream_t)stream, &ws);
    if (rc != ENEC_OK) return rc;
    return enec_compress(in, n_elems, dtype, B, params, out, out_capacity, out_bytes, ws, ENEC_STATIC_SCRATCH_BYTES, stream);
}

size_t enec_compress_bound_per_block(size_t n_elems, int dtype, uint32_t block_size)
{
    const size_t bound = enec_compress_bound(n_elems, dtype, block_size);
    if (!bound) return 0;
    const uint32_t B = block_size ? block_size : enec_default_block_size(n_elems);
    return bound + tuple_table_bytes(n_elems, B);
}

int enec_compress_per_block_batch(const enec_per_block_item *items, size_t n_items, int dtype, uint32_t group_length,
                                  void *workspace, size_t workspace_bytes, void *stream)
{
    if (!dtype_ok(dtype)) return ENEC_E_DTYPE;
    if ((!items && n_items) || !workspace || !aligned16(workspace)) return ENEC_E_ARG;
    const unsigned L = group_length ? group_length : 16u;
    if (!group_ok(L)) return ENEC_E_PARAMS;
    hipStream_t s = (hipStream_t)stream;
    // every argument is checked before anything is enqueued
    std::vector<uint32_t> Bs(n_items);
    uint64_t blocks = 0;
    for (size_t i = 0; i < n_items; ++i) {
        const enec_per_block_item &it = items[i];
        if (!it.out || (!it.in && it.n_elems) || !aligned16(it.in) || !aligned16(it.out) || it.n_elems > MAX_ELEMS)
            return ENEC_E_ARG;
        const uint32_t B = it.block_size ? it.block_size : enec_default_block_size(it.n_elems);
        if (!block_ok(B)) return ENEC_E_BLOCK;
        if (!group_fits_block(L, B)) return ENEC_E_PARAMS;
        if (it.out_capacity < enec_compress_bound_per_block(it.n_elems, dtype, B)) return ENEC_E_CAPACITY;
        if (it.out_bytes && !device_accessible(it.out_bytes)) return ENEC_E_ARG;
        Bs[i] = B;
        blocks += num_blocks(it.n_elems, B);
    }
    if (blocks > 0xFFFFFFFFull) return ENEC_E_ARG;               // block numbers are 32 bits wide
    PbCompressFn fn = pick_compress_per_block(dtype, L);
    CompressFn stream_fn = pick_compress_per_block_stream(dtype, L);
    if (!fn || !stream_fn) return ENEC_E_DTYPE;

    // Tensors of the default block size go through the kernel with deferred stores, up to MAX_BATCH to a launch, in the
    // order given; its scan words are those of enec_compress, handed out anew by every launch.  The others take the
    // kernel that places a block at once, whose ticket counters and look-back words (an even number per tensor, behind
    // the accumulators) are cleared for the call.  So does everything where the workspace has room for these words only.
    const size_t acc_words = ws_acc_words(workspace_bytes), state_words = ws_state_words(workspace_bytes);
    auto streamed = [&](size_t i) { return Bs[i] == ENEC_DEFAULT_BLOCK && items[i].n_elems != 0; };
    bool use_stream = true;
    for (size_t i = 0, in_launch = 0, groups = 0, words = 0; i < n_items; ++i) {
        if (!streamed(i)) continue;
        if (in_launch == (size_t)MAX_BATCH) in_launch = groups = words = 0;
        const size_t nb = num_blocks(items[i].n_elems, Bs[i]);
        ++in_launch;
        groups += ws_groups(nb);
        words += ws_groups(nb) + nb;
        if (groups > acc_words || acc_words + words > state_words) use_stream = false;
    }
    const size_t first = acc_words + (acc_words & 1);            // 16-byte aligned for the fill kernel
    size_t need = PB_TICKET_CLASSES * PB_TICKET_STRIDE / 2, need_all = need;      // the ticket counters, in 8-byte words
    for (size_t i = 0; i < n_items; ++i) {
        const size_t nb = num_blocks(items[i].n_elems, Bs[i]), words = nb + (nb & 1);
        need_all += words;
        if (!(use_stream && streamed(i))) need += words;
    }
    if (state_words < first + need_all) return ENEC_E_CAPACITY;
    std::vector<char> done(n_items, 0);
    if (use_stream) {
        const size_t lds = 2 * (size_t)pb_image_bytes(L) + ENEC_DEFAULT_BLOCK;
        for (size_t i = 0; i < n_items;) {
            for (; i < n_items && !streamed(i); ++i) {}
            if (i == n_items) break;
            CompressArgs a{};
            size_t word = acc_words, acc = 0;
            a.ws_ctl = reinterpret_cast<uint32_t *>(static_cast<uint8_t *>(workspace) + WS_CTL);
            a.B = ENEC_DEFAULT_BLOCK;
            a.logB = DEFAULT_LOGB;
            for (; i < n_items && a.n_items < (uint32_t)MAX_BATCH; ++i) {
                if (!streamed(i)) continue;
                fill_compress_item(a, acc, word, workspace, items[i].in, items[i].out, items[i].out_bytes, items[i].n_elems, dtype);
                CompressItem &c = a.item[a.n_items - 1];
                const size_t tuples = tuple_table_bytes(items[i].n_elems, a.B);
                c.b = 0;                              // (pads are read as zero words)
                c.mode = 0;
                c.tail_base += tuples;
                c.payload_base += tuples;
                done[i] = 1;
            }
            const unsigned resident = resident_workgroups((const void *)stream_fn, ENEC_DEFAULT_BLOCK / 64, lds);
            if (resident == 0) return ENEC_E_HIP;
            launch_compress(stream_fn, a, resident, ENEC_DEFAULT_BLOCK / 64, lds, s);
        }
    }
    if (std::find(done.begin(), done.end(), 0) == done.end()) return hipGetLastError() == hipSuccess ? ENEC_OK : ENEC_E_HIP;

    uint64_t *base = reinterpret_cast<uint64_t *>(static_cast<uint8_t *>(workspace) + WS_STATE) + first;
    const uint64_t nvec = need / 2;
    const unsigned fill_grid = (unsigned)((nvec + 255) / 256 < 1024 ? (nvec + 255) / 256 : 1024);
    fill_zero_kernel<<<fill_grid, 256, 0, s>>>(reinterpret_cast<uint4 *>(base), nvec);
    uint64_t *words = base + PB_TICKET_CLASSES * PB_TICKET_STRIDE / 2;
    uint64_t next_block = 0;        // their data blocks are numbered through, launch after launch
    for (size_t i0 = 0; i0 < n_items; ++i0) {
        if (done[i0]) continue;
        const enec_per_block_item &it0 = items[i0];
        if (it0.n_elems == 0) {     // a header and an empty table
            compress_empty_kernel<<<1, 64, 0, s>>>(static_cast<uint8_t *>(it0.out), it0.out_bytes, Bs[i0], 0, 0, 0,
                                                   (uint32_t)dtype, L | 0x100u);
            done[i0] = 1;
            continue;
        }
        // one launch for up to MAX_BATCH tensors of this block size, in the order given
        const uint32_t B = Bs[i0];
        PbCompressArgs a;
        a.ticket = reinterpret_cast<uint32_t *>(base);
        a.n_items = 0;
        a.first_block = (uint32_t)next_block;
        a.B = B; a.logB = ilog2(B);
        a.spin_limit = spin_limit();
        for (size_t i = i0; i < n_items && a.n_items < (uint32_t)MAX_BATCH; ++i) {
            const enec_per_block_item &it = items[i];
            if (done[i] || Bs[i] != B || it.n_elems == 0) continue;
            const size_t nb = num_blocks(it.n_elems, B);
            PbCompressItem &d = a.item[a.n_items++];
            d.in = it.in;
            d.out = static_cast<uint8_t *>(it.out);
            d.out_bytes = reinterpret_cast<unsigned long long *>(it.out_bytes);
            d.words = words;
            d.n_elems = it.n_elems;
            d.tuples_at = table_end(it.n_elems, B);
            d.tail_base = d.tuples_at + tuple_table_bytes(it.n_elems, B);
            d.payload_base = payload_base(it.n_elems, B, dtype) + tuple_table_bytes(it.n_elems, B);
            d.nb = (uint32_t)nb;
            d.first = (uint32_t)next_block;
            words += nb + (nb & 1);
            next_block += nb;
            done[i] = 1;
        }
        for (uint32_t i = a.n_items; i < (uint32_t)MAX_BATCH; ++i) a.item[i] = a.item[0];
        a.n_blocks = (uint32_t)(next_block - a.first_block);
        // one workgroup per data block, a thread per 64 elements (at least a wave); dynamic LDS: mask | low
        // plane | high records (at most 8 plane bits together), before that the histogram copies; behind
        // it the raw bytes of the rows that do not wait in registers
        const unsigned threads = B / 64 < 64 ? 64 : B / 64;
        const size_t image = (size_t)B / (8 * L) + (size_t)B, hist = (size_t)PB_HIST_COPIES * PB_HIST_STRIDE * 4;
        const size_t lds = (image > hist ? image : hist) + 15 & ~(size_t)15;
        a.park_at = (uint32_t)lds;
        hipLaunchKernelGGL(fn, dim3(a.n_blocks), dim3(threads), lds + (size_t)(8 - PB_SM_REG_ROWS) * threads * 8, s, a);
    }
    return hipGetLastError() == hipSuccess ? ENEC_OK : ENEC_E_HIP;
}

int enec_compress_per_block(const void *in, size_t n_elems, int dtype, uint32_t block_size, uint32_t group_length,
                            void *out, size_t out_capacity, uint64_t *out_bytes, void *workspace,
                            size_t workspace_bytes, void *stream)
{
    enec_per_block_item it;
    it.in = in;
    it.n_elems = n_elems;
    it.block_size = block_size;
    it.out = out;
    it.out_capacity = out_capacity;
    it.out_bytes = out_bytes;
    return enec_compress_per_block_batch(&it, 1, dtype, group_length, workspace, workspace_bytes, stream);
}

int enec_decompress_batch(const enec_decompress_item *items, size_t n_items, void *stream)
{
    hipStream_t s = (hipStream_t)stream;
    if (!items) return ENEC_E_ARG;
    std::vector<Header> hdr(n_items);
    for (size_t i = 0; i < n_items; ++i) {
        const enec_decompress_item &it = items[i];
        if (!it.in || !it.host_header || (!it.out && it.n_elems) || !aligned16(it.in) || !aligned16(it.out) ||
            ((uintptr_t)it.status & 3))
            return ENEC_E_ARG;
        if (it.status && !device_accessible(it.status)) return ENEC_E_ARG;
        Header &h = hdr[i];
        int rc = parse_header(it.host_header, &h);
        if (rc != ENEC_OK) return rc;
        if (h.status != ENEC_OK || h.n_elems != it.n_elems || !block_ok(h.B) || it.n_elems > MAX_ELEMS ||
            h.nb != num_blocks(it.n_elems, h.B) || !group_fits_block(h.prm.L, h.B) || h.total > it.in_bytes)
            return ENEC_E_FORMAT;
        if (h.per_block) {
            if (h.prm.n != 0 || h.prm.m != 0 || h.prm.b != 0 ||
                h.total < payload_base(it.n_elems, h.B, h.dtype) + tuple_table_bytes(it.n_elems, h.B))
                return ENEC_E_FORMAT;
        } else if (h.prm.n < 1 || h.prm.n > exp_bits(h.dtype) || h.prm.m > h.prm.n ||
                   h.prm.b >= (1u << exp_bits(h.dtype)) || h.total < payload_base(it.n_elems, h.B, h.dtype)) {
            return ENEC_E_FORMAT;
        }
    }
    // Streams of one element format, group length and block size share a launch (up to MAX_BATCH each),
    // whether they have one tuple or one tuple per block and whatever the tuples are.  A stream of at most JOIN blocks
    // joins a launch of larger blocks too: each of its blocks takes the place of a large one, 8 us of one of the device's
    // 1024 places, where a launch of their own takes 4 us of all of them.  A decoder layer with its two norm vectors, us:
    // hidden size 512 10.9 -> 7.2, 1024 12.5 -> 8.7, 2048 35.9 -> 31.8, 4096 120.9 -> 118.1.
    // The streams of the launch's block size are in it first: sixteen small ones ahead of a large one would else take all
    // places of a launch with its threads and LDS, and leave it to a launch of its own.  Of a smaller size as many join as
    // make one launch less for that size; fewer would save no launch and move one more to the instances for mixed sizes
    // (40 vectors of three sizes 18.9 -> 18.2 us, as fp32 26.2 -> 25.2; sixteen vectors and a matrix 13.4 -> 12.6).
    constexpr uint32_t JOIN = 16;
    constexpr uint8_t NONE = 255;                            // an empty stream, or one that a launch has taken
    struct Kind { uint8_t like, size; };                     // element format and group length; block size, 2048 .. 32768 -> 0 .. 4
    std::vector<Kind> kind(n_items);
    struct { uint32_t all, few; } left[9][5] = {};           // streams that no launch has taken yet, and those of few blocks
    for (size_t j = 0; j < n_items; ++j) {
        const Header &h = hdr[j];
        kind[j].like = h.nb == 0 ? NONE : (uint8_t)(3 * h.dtype + __builtin_ctz(h.prm.L) - 3);
        kind[j].size = (uint8_t)(__builtin_ctz(h.B) - 11);
        if (h.nb == 0) continue;
        auto &l = left[kind[j].like][kind[j].size];
        ++l.all;
        l.few += h.nb <= JOIN;
    }
    for (size_t i = 0; i < n_items;) {
        if (kind[i].like == NONE) { ++i; continue; }
        const Header &h0 = hdr[i];
        const uint8_t like = kind[i].like;
        auto &l = left[like];
        unsigned c = kind[i].size;
        if (h0.nb <= JOIN)
            for (c = 4; l[c].all == 0; --c) {}
        const uint32_t B = 2048u << c;
        uint32_t take[5] = {}, places = MAX_BATCH;           // streams of each block size that this launch takes
        take[c] = std::min(l[c].all, places);
        places -= take[c];
        while (c-- > 0 && places != 0) {
            const uint32_t last = l[c].all ? (l[c].all - 1) % MAX_BATCH + 1 : 0;      // what the last launch of this size would hold
            if (last <= l[c].few && last <= places) { take[c] = last; places -= last; }
        }
        const unsigned threads = B / 64 < 64 ? 64 : B / 64;
        DecompressArgs a;
        a.B = B;
        a.logB = ilog2(B);
        bool mixed = false;
        uint32_t items_in = 0;
        uint64_t blocks = 0;
        size_t packed = 0;       // the packed part of the widest block of the launch: mask | low plane | high records | padding
        for (size_t j = i; j < n_items && items_in < MAX_BATCH - places; ++j) {
            if (kind[j].like != like || take[kind[j].size] == 0) continue;
            const Header &h = hdr[j];
            if ((h.B != B && h.nb > JOIN) || (blocks + h.nb) * threads > 0xFFFFFFFFull) continue;   // a grid has fewer than 2^32 threads
            kind[j].like = NONE;
            --take[kind[j].size];
            --l[kind[j].size].all;
            l[kind[j].size].few -= h.nb <= JOIN;
            const size_t tuples = h.per_block ? tuple_table_bytes(items[j].n_elems, h.B) : 0;
            a.first[items_in] = (uint32_t)blocks;
            DecompressItem &d = a.item[items_in++];
            d.in = static_cast<const uint8_t *>(items[j].in);
            d.out = items[j].out;
            d.n_elems = items[j].n_elems;
            d.tuples_at = h.per_block ? table_end(d.n_elems, h.B) : 24;
            d.tuple_stride = h.per_block ? 4u : 0u;
            d.tail_base = table_end(d.n_elems, h.B) + tuples;
            d.payload_base = payload_base(d.n_elems, h.B, h.dtype) + tuples;
            d.payload_bytes = h.total - d.payload_base;
            d.status = items[j].status;
            d.logB = 11u + kind[j].size;
            mixed |= h.B != B;
            std::memcpy(d.hdr, items[j].host_header, sizeof d.hdr);
            const uint32_t bits = h.per_block ? 8u : h.prm.n + (h.dtype == ENEC_FP16 ? 3u : 0u);
            packed = std::max(packed, (size_t)h.B / (8 * h.prm.L) + (size_t)bits * h.B / 8 + 16);
            blocks += h.nb;
        }
        for (uint32_t j = items_in; j < (uint32_t)MAX_BATCH; ++j) {
            a.first[j] = 0xFFFFFFFFu;
            a.item[j] = a.item[0];
        }
        DecompressFn fn = items_in == 1 && !mixed ? pick_decompress_one(h0.dtype, h0.prm.L) : pick_decompress(h0.dtype, h0.prm.L, mixed);
        if (!fn) return ENEC_E_FORMAT;
        size_t lds = packed + (h0.dtype == ENEC_FP32 ? 16 * threads : 0);
        if (h0.dtype != ENEC_FP32 && lds < decompress_lds_floor(B)) lds = decompress_lds_floor(B);
        a.turn_at = (uint32_t)packed;
        hipLaunchKernelGGL(fn, dim3((unsigned)blocks), dim3(threads), lds, s, a);
    }
    return hipGetLastError() == hipSuccess ? ENEC_OK : ENEC_E_HIP;
}

int enec_decompress_with_header(const void *in, size_t in_bytes, const void *host_header, void *out,
                                size_t n_elems, uint32_t *status, void *stream)
{
    enec_decompress_item it;
    it.in = in; it.in_bytes = in_bytes; it.host_header = host_header; it.out = out; it.n_elems = n_elems;
    it.status = status;
    return enec_decompress_batch(&it, 1, stream);
}

int enec_decompress(const void *in, size_t in_bytes, void *out, size_t n_elems, void *stream)
{
    if (!in || !aligned16(in)) return ENEC_E_ARG;
    if (in_bytes < ENEC_HEADER_BYTES) return ENEC_E_FORMAT;
    uint8_t hdr[ENEC_HEADER_BYTES];
    hipStream_t s = (hipStream_t)stream;
    if (hipMemcpyAsync(hdr, in, sizeof hdr, hipMemcpyDeviceToHost, s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess) {
        (void)hipGetLastError();
        return ENEC_E_HIP;
    }
    return enec_decompress_with_header(in, in_bytes, hdr, out, n_elems, nullptr, stream);
}

int enec_stream_info(const void *host_header, enec_params *params, uint64_t *n_elems,
                     uint32_t *block_size, uint64_t *total_bytes, int *dtype, uint32_t *status)
{
    if (!host_header) return ENEC_E_ARG;
    Header h;
    int rc = parse_header(host_header, &h);
    if (rc != ENEC_OK) return rc;
    if (params) *params = h.prm;
    if (n_elems) *n_elems = h.n_elems;
    if (block_size) *block_size = h.B;
    if (total_bytes) *total_bytes = h.total;
    if (dtype) *dtype = h.dtype;
    if (status) *status = h.status;
    return ENEC_OK;
}

int enec_copy(void *dst, const void *src, size_t bytes, void *stream)
{
    if (!dst || !src || !aligned16(dst) || !aligned16(src) || (bytes & 15)) return ENEC_E_ARG;
    const uint64_t nvec = bytes / 16;
    if (nvec == 0) return ENEC_OK;
    uint64_t want = (nvec + 255) / 256;
    const unsigned grid = (unsigned)(want > 8192 ? 8192 : want);
    copy_kernel<<<grid, 256, 0, (hipStream_t)stream>>>(static_cast<uint4 *>(dst), static_cast<const uint4 *>(src), nvec);
    return hipGetLastError() == hipSuccess ? ENEC_OK : ENEC_E_HIP;
}

}  // extern "C"

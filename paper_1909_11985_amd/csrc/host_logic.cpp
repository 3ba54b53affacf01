// Host-side integer logic and model tables: shard assignment (sections 3.1
// and 4.3 of the paper), He initialisation, and the layer lists of the four
// model families.  No GPU code here.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <thread>

#include "graph.h"

#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
#include <immintrin.h>
#endif

namespace edl {

// ---------------------------------------------------------------- errors
static thread_local char g_err[512] = "";

void set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}
const char* get_error() { return g_err; }

// ---------------------------------------------------------------- generator
// SplitMix64 used as a counter-based generator: draw j of a stream is the
// finaliser applied to key + (j+1)*golden.
static const uint64_t kGolden = 0x9E3779B97F4A7C15ull;
static const uint64_t kInitKey = 0xD1B54A32D192ED03ull;

static inline uint64_t mix64(uint64_t key, uint64_t j) {
    uint64_t z = key + (j + 1) * kGolden;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}
uint64_t splitmix64_at(uint64_t key, uint64_t j) { return mix64(key, j); }

// The leader's random permutation of section 4.3, one per epoch: Fisher-Yates
// from the last position down, partner index = high 64 bits of draw*(i+1).
// A position is final once the walk has passed it, so a caller that wants the
// entries from `from` on stops there (the mini-batches of an epoch: half the
// walk on average).
//
// Partners are drawn kAhead at a time and their cache lines asked for before the swaps that need them.  Below 2^32
// entries the product's high half is two 32x32 products, so that the draws vectorise (the build targets plain x86-64:
// the loop is compiled for wider vectors as well and chosen by what the machine has).
constexpr int kAhead = 64;

#define EDL_DRAW_PARTNERS                                                                            \
    for (int k = 0; k < kAhead; ++k) {                                                               \
        const uint64_t r = mix64(key, draw + (uint64_t)k), m = (uint64_t)(i + 1) - (uint64_t)k; \
        partner[k] = (uint32_t)(((r >> 32) * (m & 0xffffffffu) + (((r & 0xffffffffu) * (m & 0xffffffffu)) >> 32)) >> 32); \
    }
static void draw_partners_plain(uint64_t key, uint64_t draw, int64_t i, uint32_t* partner) { EDL_DRAW_PARTNERS }
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
__attribute__((target("avx2"))) static void draw_partners_avx2(uint64_t key, uint64_t draw, int64_t i, uint32_t* partner) { EDL_DRAW_PARTNERS }
__attribute__((target("avx512f,avx512dq,avx512vl"))) static void draw_partners_avx512(uint64_t key, uint64_t draw, int64_t i, uint32_t* partner) { EDL_DRAW_PARTNERS }
#endif
#undef EDL_DRAW_PARTNERS

typedef void (*DrawPartners)(uint64_t, uint64_t, int64_t, uint32_t*);
static DrawPartners pick_draw_partners() {
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
    __builtin_cpu_init();
    if (__builtin_cpu_supports("avx512f") && __builtin_cpu_supports("avx512dq") && __builtin_cpu_supports("avx512vl")) return draw_partners_avx512;
    if (__builtin_cpu_supports("avx2")) return draw_partners_avx2;
#endif
    return draw_partners_plain;
}

// Draws kAhead partners as above and sifts them: bit t of the result is clear where partner[t] is none of the locations that
// the sieve holds (it may be set for others: 250 locations let one in 2,000 through).  Five tables of 1,024 bits stay in
// registers, looked up by byte permutes; a location has a bit in each, found by five fields of it and of its product with an odd
// constant.
struct alignas(64) Sieve {
    unsigned char bits[5][128];
    void add(uint32_t x) {
        const unsigned char bit = (unsigned char)(1u << (x & 7));
        const uint32_t h = x * 0x9E3779B1u;
        bits[0][(x >> 3) & 127] |= bit;
        bits[1][(x >> 10) & 127] |= bit;
        bits[2][(h >> 25) & 127] |= bit;
        bits[3][(h >> 18) & 127] |= bit;
        bits[4][(h >> 11) & 127] |= bit;
    }
};
typedef uint64_t (*SiftPartners)(uint64_t, uint64_t, int64_t, uint32_t*, const Sieve&);
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
__attribute__((target("avx512f,avx512dq,avx512vl,avx512bw,avx512vbmi"))) static uint64_t sift_partners_avx512(uint64_t key, uint64_t draw, int64_t i,
                                                                                                             uint32_t* partner, const Sieve& sieve) {
    draw_partners_avx512(key, draw, i, partner);
    __m512i table[10];
    for (int t = 0; t < 10; ++t) table[t] = _mm512_load_si512((const char*)sieve.bits + 64 * t);
    const __m512i one = _mm512_set1_epi32(1), seven = _mm512_set1_epi32(7), odd = _mm512_set1_epi32((int)0x9E3779B1u);
    uint64_t hits = 0;
    for (int t = 0; t < kAhead; t += 16) {
        // (of each lane's four bytes the lowest counts: the bit asked for lies there)
        const __m512i x = _mm512_loadu_si512(partner + t), bit = _mm512_sllv_epi32(one, _mm512_and_si512(x, seven)), h = _mm512_mullo_epi32(x, odd);
        __m512i in = _mm512_permutex2var_epi8(table[0], _mm512_srli_epi32(x, 3), table[1]);
        in = _mm512_and_si512(in, _mm512_permutex2var_epi8(table[2], _mm512_srli_epi32(x, 10), table[3]));
        in = _mm512_and_si512(in, _mm512_permutex2var_epi8(table[4], _mm512_srli_epi32(h, 25), table[5]));
        in = _mm512_and_si512(in, _mm512_permutex2var_epi8(table[6], _mm512_srli_epi32(h, 18), table[7]));
        in = _mm512_and_si512(in, _mm512_permutex2var_epi8(table[8], _mm512_srli_epi32(h, 11), table[9]));
        hits |= (uint64_t)_mm512_test_epi32_mask(in, bit) << t;
    }
    return hits;
}
#endif
static SiftPartners pick_sift_partners() {
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
    __builtin_cpu_init();
    if (__builtin_cpu_supports("avx512f") && __builtin_cpu_supports("avx512dq") && __builtin_cpu_supports("avx512vl") &&
        __builtin_cpu_supports("avx512bw") && __builtin_cpu_supports("avx512vbmi")) return sift_partners_avx512;
#endif
    return nullptr;
}
static const SiftPartners& sift_partners() {
    static const SiftPartners f = pick_sift_partners();
    return f;
}
constexpr int64_t kSieved = 400;       // entries that the sieve still tells apart: a third of its bits set, one draw in 280 let through

template <typename I>
static void shuffle_down_to(uint64_t key, int64_t N, int64_t from, I* perm) {
    static const DrawPartners draw_partners = pick_draw_partners();
    for (int64_t i = 0; i < N; ++i) perm[i] = (I)i;
    const int64_t last = std::max<int64_t>(from, 1);
    uint64_t draw = 0;
    int64_t i = N - 1;
    if (N <= (int64_t)0xffffffffll) {
        uint32_t partner[kAhead];
        while (i - kAhead >= last) {
            draw_partners(key, draw, i, partner);
            for (int k = 0; k < kAhead; ++k) __builtin_prefetch(perm + partner[k], 1);
            for (int k = 0; k < kAhead; ++k, --i) {
                const I t = perm[i];
                perm[i] = perm[partner[k]];
                perm[partner[k]] = t;
            }
            draw += kAhead;
        }
    }
    for (; i >= last; --i) {
        const uint64_t r = mix64(key, draw++);
        const uint64_t j = (uint64_t)(((unsigned __int128)r * (unsigned __int128)(uint64_t)(i + 1)) >> 64);
        const I t = perm[i];
        perm[i] = perm[j];
        perm[j] = t;
    }
}

static uint64_t epoch_key(uint64_t seed, int64_t epoch) { return seed ^ (kGolden * (uint64_t)(epoch + 1)); }

void epoch_permutation(uint64_t seed, int64_t epoch, int64_t N, std::vector<int64_t>& perm) {
    perm.resize((size_t)N);
    shuffle_down_to<int64_t>(epoch_key(seed, epoch), N, 0, perm.data());
}

// Entries [from, from + count) of it.
//
// The walk moves whole entries to find a few.  An entry can be followed backwards instead: position i ends with what
// location j_i held when the walk came to i, and what a location x holds then was put there by the last step before, the
// smallest k > i with j_k = x, from location k as it was at step k; with no such step it holds x.  So the steps are looked at
// from `from` upwards with the locations that are being followed, `count` of them: a step whose partner is one of them moves
// that entry to location k, and nearly all steps (all but count / k of them) are none of their business.  A table of
// bits that stays in the first-level cache says which partners may matter; the steps left over are looked up exactly.
// Nothing is written per step and no array of N entries is laid out.
// 1.2 million samples, mini-batches of 250, the epoch's first / middle / last one on the host of an MI355X: walked 1,028 / 553
// / 54 us, followed 700 / 306 / 5.
namespace {
class Followed {
public:
    Followed(int64_t count) {
        size_t slots = 16;
        while (slots < (size_t)count * 4) slots *= 2;
        key_.assign(slots, kNone);
        entry_.resize(slots);
        where_.assign((size_t)count, 0);
        maybe_.assign(kFilter / 64, 0);
        std::memset(&sieve_, 0, sizeof(sieve_));
    }
    // entry e is now followed at location x
    void put(uint32_t x, uint32_t e) {
        size_t s = slot(x);
        while (key_[s] != kNone) s = (s + 1) & (key_.size() - 1);
        key_[s] = x;
        entry_[s] = e;
        where_[e] = x;
        mark(x);
    }
    bool may_be(uint32_t x) const { return (maybe_[(x & (kFilter - 1)) / 64] >> (x & 63)) & 1; }
    const uint64_t* filter() const { return maybe_.data(); }
    const Sieve& sieve() const { return sieve_; }
    // the step k with partner x: an entry followed at x comes from location k
    bool step(uint32_t x, uint32_t k) {
        size_t s = slot(x);
        while (key_[s] != x) {
            if (key_[s] == kNone) return false;
            s = (s + 1) & (key_.size() - 1);
        }
        const uint32_t e = entry_[s];
        // take the slot out: later ones of the same run move up
        for (size_t hole = s;;) {
            key_[hole] = kNone;
            size_t t = hole;
            for (;;) {
                t = (t + 1) & (key_.size() - 1);
                if (key_[t] == kNone) goto closed;
                const size_t home = slot(key_[t]);
                if (((t - home) & (key_.size() - 1)) >= ((t - hole) & (key_.size() - 1))) break;
            }
            key_[hole] = key_[t];
            entry_[hole] = entry_[t];
            hole = t;
        }
    closed:
        put(k, e);
        // bits of locations left behind stay set; many of them would let too many steps through
        if (++sifted_ == 48) {
            sifted_ = 0;
            std::memset(&sieve_, 0, sizeof(sieve_));
            for (uint32_t x : where_) sieve_.add(x);
        }
        if (++moved_ == 256 + where_.size() / 2) {
            moved_ = 0;
            std::fill(maybe_.begin(), maybe_.end(), 0);
            for (uint32_t x : key_)
                if (x != kNone) mark(x);
        }
        return true;
    }
    uint32_t where(size_t e) const { return where_[e]; }
    static constexpr uint32_t kFilter = 1u << 18;       // bits: 32 KB

private:
    static constexpr uint32_t kNone = 0xffffffffu;      // (locations are below N < 2^32 - 1)
    void mark(uint32_t x) {
        maybe_[(x & (kFilter - 1)) / 64] |= 1ull << (x & 63);
        sieve_.add(x);
    }
    size_t slot(uint32_t x) const { return (size_t)((x * 0x9E3779B1u) >> 7) & (key_.size() - 1); }
    std::vector<uint32_t> key_, entry_, where_;
    std::vector<uint64_t> maybe_;
    Sieve sieve_;
    uint32_t moved_ = 0, sifted_ = 0;
};
}  // namespace

static void follow_entries(uint64_t key, int64_t N, int64_t from, int64_t count, int64_t* out) {
    static const DrawPartners draw_partners = pick_draw_partners();
    Followed f(count);
    int64_t k = from;
    for (; k < from + count; ++k) {
        uint32_t j = 0;
        if (k > 0) {
            const uint64_t r = mix64(key, (uint64_t)(N - 1 - k));
            j = (uint32_t)(((unsigned __int128)r * (unsigned __int128)(uint64_t)(k + 1)) >> 64);
            f.step(j, (uint32_t)k);
        }
        f.put(j, (uint32_t)(k - from));
    }
    uint32_t partner[kAhead];
    if (const SiftPartners sift = count <= kSieved ? sift_partners() : nullptr)
        for (; k + kAhead <= N; k += kAhead) {
            uint64_t hits = sift(key, (uint64_t)(N - k - kAhead), k + kAhead - 1, partner, f.sieve());
            while (hits != 0) {       // (the last of them is the first step)
                const int t = 63 - __builtin_clzll(hits);
                hits &= ~(1ull << t);
                if (!f.may_be(partner[t]) || !f.step(partner[t], (uint32_t)(k + kAhead - 1 - t))) continue;
                // an entry has moved: the rest of the steps have been sifted for where it was
                for (int u = t - 1; u >= 0; --u)
                    if (f.may_be(partner[u])) f.step(partner[u], (uint32_t)(k + kAhead - 1 - u));
                break;
            }
        }
    for (; k + kAhead <= N; k += kAhead) {
        // partner[t] belongs to step k + kAhead - 1 - t
        draw_partners(key, (uint64_t)(N - k - kAhead), k + kAhead - 1, partner);
        const uint64_t* const maybe = f.filter();
        for (int t0 = kAhead - 8; t0 >= 0; t0 -= 8) {
            uint64_t any = 0;
            for (int t = 0; t < 8; ++t) any |= maybe[(partner[t0 + t] & (Followed::kFilter - 1)) / 64] >> (partner[t0 + t] & 63);
            if ((any & 1) == 0) continue;
            for (int t = t0 + 7; t >= t0; --t)
                if (f.may_be(partner[t])) f.step(partner[t], (uint32_t)(k + kAhead - 1 - t));
        }
    }
    for (; k < N; ++k) {
        const uint64_t r = mix64(key, (uint64_t)(N - 1 - k));
        f.step((uint32_t)(((unsigned __int128)r * (unsigned __int128)(uint64_t)(k + 1)) >> 64), (uint32_t)k);
    }
    for (int64_t e = 0; e < count; ++e) out[e] = (int64_t)f.where((size_t)e);
}

void epoch_permutation_slice(uint64_t seed, int64_t epoch, int64_t N, int64_t from, int64_t count, int64_t* out) {
    // ns on the host of an MI355X: following costs 1,000 for its tables, 3 an entry, 25 every time an entry moves (ln(N / from) times each),
    // 0.45 a step and 20 for each step that the table of bits lets through (2^18 bits: count / 2^18 of them, and more while bits of
    // left locations stay set); the walk 0.047 an entry for its array and 0.71 a step.  Small data sets and mini-batches that are a
    // large part of theirs are walked.  us, walked / followed: 50,048 samples in mini-batches of 128, the first 42 / 66, the last
    // quarter's 15 / 11; 500,000 in 1,000, the first 371 / 507, the last 1% 28 / 9; 2.5 million in 4,000, the first 2,029 / 3,153, the last
    // 10% 310 / 192; in 250, the first 2,018 / 1,303.  Over 2,000 to 5 million samples in mini-batches of 1 to 30,000 the rule's choice
    // takes 0.5% longer than the better one in the mean, 10% at most where it follows.
    // With the sieve (up to kSieved entries, 512-bit vectors with byte permutes): 0.28 a step and 36 a move.  us, before / with it:
    // 1.2 million in 250, the first 679 / 433, the middle one 294 / 174; in 400 723 / 563 and 307 / 202; 2.5 million in 250 1,326 / 803
    // and 609 / 351; 100,000 in 100 81 / 53 and 28 / 20.
    const double steps = (double)(N - from), entries = (double)count;
    const bool sieved = count <= kSieved && sift_partners() != nullptr;
    const double follow = 1000.0 + 3.0 * entries + (sieved ? 36.0 : 25.0) * entries * std::log((double)N / (double)(from + count)) +
                          (sieved ? 2.0 : 20.0) * steps * entries / (double)(1 << 18);
    if (N < (int64_t)0xffffffffll && follow < 0.047 * (double)N + (sieved ? 0.42 : 0.26) * steps) {
        follow_entries(epoch_key(seed, epoch), N, from, count, out);
        return;
    }
    // The walk: bound by its random accesses and, for large data sets, by the pages of a fresh work array: 32-bit entries halve
    // the array and each thread keeps its own from call to call (released above kKeptEntries).
    constexpr int64_t kKeptEntries = 4 << 20;
    if (N > (int64_t)0xffffffffll) {
        std::vector<int64_t> perm((size_t)N);
        shuffle_down_to<int64_t>(epoch_key(seed, epoch), N, from, perm.data());
        std::copy(perm.begin() + from, perm.begin() + from + count, out);
        return;
    }
    static thread_local std::vector<uint32_t> kept;
    std::vector<uint32_t> own;
    std::vector<uint32_t>& perm = N <= kKeptEntries ? kept : own;
    if ((int64_t)perm.size() < N) perm.resize((size_t)N);
    shuffle_down_to<uint32_t>(epoch_key(seed, epoch), N, from, perm.data());
    for (int64_t i = 0; i < count; ++i) out[i] = (int64_t)perm[(size_t)(from + i)];
}

// He-normal weights by Box-Muller on the counter-based draws, one stream per
// parameter tensor (keyed by the tensor's position in the flat vector).
void he_init(const Graph& g, uint64_t seed, float* out) {
    for (size_t t = 0; t < g.params.size(); ++t) {
        const ParamTensor& pt = g.params[t];
        float* dst = out + pt.off;
        if (pt.fan_in == 0) {
            const float fill = pt.is_gamma ? 1.0f : 0.0f;
            for (int64_t i = 0; i < pt.size; ++i) dst[i] = fill;
            continue;
        }
        const uint64_t key = seed ^ (kInitKey * (uint64_t)(t + 1));
        const double sd = std::sqrt(2.0 / (double)pt.fan_in);
        const double two_pi = 2.0 * 3.14159265358979323846;
        const int64_t pairs = (pt.size + 1) / 2;
        const int64_t size = pt.size;
        auto fill = [=](int64_t q0, int64_t q1) {
            for (int64_t q = q0; q < q1; ++q) {
                const uint64_t r1 = splitmix64_at(key, (uint64_t)(2 * q));
                const uint64_t r2 = splitmix64_at(key, (uint64_t)(2 * q + 1));
                const double u1 = ((double)(r1 >> 11) + 1.0) * 0x1.0p-53;
                const double u2 = (double)(r2 >> 11) * 0x1.0p-53;
                const double rad = std::sqrt(-2.0 * std::log(u1));
                const double ang = two_pi * u2;
                dst[2 * q] = (float)(rad * std::cos(ang) * sd);
                if (2 * q + 1 < size) dst[2 * q + 1] = (float)(rad * std::sin(ang) * sd);
            }
        };
        unsigned nt = std::thread::hardware_concurrency();
        if (nt == 0) nt = 1;
        if (nt > 16) nt = 16;
        if (pairs < (1 << 16) || nt == 1) {
            fill(0, pairs);
        } else {
            std::vector<std::thread> pool;
            const int64_t per = (pairs + nt - 1) / nt;
            for (unsigned i = 0; i < nt; ++i) {
                const int64_t a = (int64_t)i * per, b = a + per < pairs ? a + per : pairs;
                if (a < b) pool.emplace_back(fill, a, b);
            }
            for (auto& th : pool) th.join();
        }
    }
}

// ---------------------------------------------------------------- graph
static int out_extent(int in, int k, int stride, int pad) { return (in + 2 * pad - k) / stride + 1; }

int Graph::add_tensor(int H, int W, int C) {
    Tensor t;
    t.H = H; t.W = W; t.C = C;
    tensors.push_back(t);
    return (int)tensors.size() - 1;
}

int Graph::conv(int x, int K, int R, int stride, int pad, bool bias, bool relu, const std::string& name) {
    const Tensor tx = tensors[(size_t)x];
    Op op;
    op.kind = OP_CONV; op.x = x; op.K = K; op.R = R; op.S = R; op.stride = stride; op.pad = pad;
    op.bias = bias; op.relu = relu; op.name = name;
    op.w_off = P;
    const int64_t wsize = (int64_t)K * R * R * tx.C;
    params.push_back({name + ".w", P, wsize, (int64_t)tx.C * R * R, false});
    P += wsize;
    if (bias) {
        op.b_off = P;
        params.push_back({name + ".b", P, K, 0, false});
        P += K;
    }
    op.y = add_tensor(out_extent(tx.H, R, stride, pad), out_extent(tx.W, R, stride, pad), K);
    ops.push_back(op);
    return op.y;
}

int Graph::bn(int x, bool relu, int res, const std::string& name) {
    const Tensor tx = tensors[(size_t)x];
    Op op;
    op.kind = OP_BN; op.x = x; op.res = res; op.relu = relu; op.K = tx.C; op.name = name;
    op.w_off = P; op.b_off = P + tx.C; op.run_off = R;
    params.push_back({name + ".g", P, tx.C, 0, true});
    params.push_back({name + ".b", P + tx.C, tx.C, 0, false});
    P += 2 * tx.C;
    R += 2 * tx.C;
    op.y = add_tensor(tx.H, tx.W, tx.C);
    ops.push_back(op);
    return op.y;
}

int Graph::maxpool(int x, int k, int stride, int pad) {
    const Tensor tx = tensors[(size_t)x];
    Op op;
    op.kind = OP_MAXPOOL; op.x = x; op.R = k; op.S = k; op.stride = stride; op.pad = pad;
    op.y = add_tensor(out_extent(tx.H, k, stride, pad), out_extent(tx.W, k, stride, pad), tx.C);
    ops.push_back(op);
    return op.y;
}

int Graph::gavgpool(int x) {
    const Tensor tx = tensors[(size_t)x];
    Op op;
    op.kind = OP_GAVGPOOL; op.x = x;
    op.y = add_tensor(1, 1, tx.C);
    ops.push_back(op);
    return op.y;
}

int Graph::flatten(int x) {
    const Tensor tx = tensors[(size_t)x];
    const int y = add_tensor(1, 1, tx.H * tx.W * tx.C);
    tensors[(size_t)y].alias_of = tensors[(size_t)x].alias_of >= 0 ? tensors[(size_t)x].alias_of : x;
    return y;
}

void Graph::loss(int x) {
    Op op;
    op.kind = OP_LOSS; op.x = x;
    ops.push_back(op);
    logits = x;
    tensors[(size_t)x].fp32 = true;
    classes = tensors[(size_t)x].C;
}

// 2 flops per multiply-add, forward + input-gradient + weight-gradient
// contractions; the first layer has no input gradient.
double Graph::flops_per_sample() const {
    double f = 0;
    for (const Op& op : ops) {
        if (op.kind != OP_CONV) continue;
        const Tensor& ty = tensors[(size_t)op.y];
        const Tensor& tx = tensors[(size_t)op.x];
        const double macs = (double)ty.H * ty.W * op.K * op.R * op.S * tx.C;
        const bool first = (op.x == 0) || (tensors[(size_t)op.x].alias_of == 0);
        f += 2.0 * macs * (first ? 2.0 : 3.0);
    }
    return f;
}

static int pick(int v, int dflt) { return v > 0 ? v : dflt; }

static void build_mlp(const edl_config& c, Graph& g) {
    const int H = pick(c.H, 1), W = pick(c.W, 1), C = pick(c.C, 784);
    const int h1 = pick(c.arch[0], 256), h2 = pick(c.arch[1], 256), classes = pick(c.classes, 10);
    int t = g.flatten(g.add_tensor(H, W, C));
    t = g.conv(t, h1, 1, 1, 0, true, true, "fc1");
    t = g.conv(t, h2, 1, 1, 0, true, true, "fc2");
    t = g.conv(t, classes, 1, 1, 0, true, false, "fc3");
    g.loss(t);
}

static std::string blk(int stage, int block) {
    char buf[32];
    snprintf(buf, sizeof(buf), "s%d.b%d", stage, block);
    return buf;
}

// CIFAR-style residual net: 3x3 stem, `stages` stages of `blocks` basic blocks,
// width doubling and stride 2 at each stage change, where the shortcut is a
// strided 1x1 projection with its own batch norm.
static void build_resnet20(const edl_config& c, Graph& g) {
    const int H = pick(c.H, 32), W = pick(c.W, 32), C = pick(c.C, 3), classes = pick(c.classes, 10);
    const int w0 = pick(c.arch[0], 16), stages = pick(c.arch[1], 3), blocks = pick(c.arch[2], 3);
    int t = g.conv(g.add_tensor(H, W, C), w0, 3, 1, 1, false, false, "stem.conv");
    t = g.bn(t, true, -1, "stem.bn");
    int cin = w0;
    for (int s = 0; s < stages; ++s) {
        const int width = w0 << s;
        for (int b = 0; b < blocks; ++b) {
            const int stride = (s > 0 && b == 0) ? 2 : 1;
            const std::string nm = blk(s + 1, b + 1);
            int u = g.conv(t, width, 3, stride, 1, false, false, nm + ".conv1");
            u = g.bn(u, true, -1, nm + ".bn1");
            u = g.conv(u, width, 3, 1, 1, false, false, nm + ".conv2");
            int sc = t;
            if (stride != 1 || cin != width) {
                sc = g.conv(t, width, 1, stride, 0, false, false, nm + ".proj");
                sc = g.bn(sc, false, -1, nm + ".projbn");
            }
            t = g.bn(u, true, sc, nm + ".bn2");
            cin = width;
        }
    }
    t = g.gavgpool(t);
    t = g.conv(t, classes, 1, 1, 0, true, false, "fc");
    g.loss(t);
}

// Bottleneck residual net: 7x7/2 stem, 3x3/2 max pool, stages of
// 1x1 - 3x3 - 1x1 blocks (the 3x3 carries the stride), projection shortcut on
// the first block of every stage.
static void build_resnet50(const edl_config& c, Graph& g) {
    const int H = pick(c.H, 224), W = pick(c.W, 224), C = pick(c.C, 3), classes = pick(c.classes, 1000);
    const int base = pick(c.arch[0], 64);
    int nb[4] = {3, 4, 6, 3};
    if (c.arch[1] > 0) for (int i = 0; i < 4; ++i) nb[i] = c.arch[1 + i];
    int t = g.conv(g.add_tensor(H, W, C), base, 7, 2, 3, false, false, "stem.conv");
    t = g.bn(t, true, -1, "stem.bn");
    t = g.maxpool(t, 3, 2, 1);
    for (int s = 0; s < 4 && nb[s] > 0; ++s) {
        const int width = base << s;
        for (int b = 0; b < nb[s]; ++b) {
            const int stride = (s > 0 && b == 0) ? 2 : 1;
            const std::string nm = blk(s + 1, b + 1);
            int u = g.conv(t, width, 1, 1, 0, false, false, nm + ".conv1");
            u = g.bn(u, true, -1, nm + ".bn1");
            u = g.conv(u, width, 3, stride, 1, false, false, nm + ".conv2");
            u = g.bn(u, true, -1, nm + ".bn2");
            u = g.conv(u, 4 * width, 1, 1, 0, false, false, nm + ".conv3");
            int sc = t;
            if (b == 0) {
                sc = g.conv(t, 4 * width, 1, stride, 0, false, false, nm + ".proj");
                sc = g.bn(sc, false, -1, nm + ".projbn");
            }
            t = g.bn(u, true, sc, nm + ".bn3");
        }
    }
    t = g.gavgpool(t);
    t = g.conv(t, classes, 1, 1, 0, true, false, "fc");
    g.loss(t);
}

// Biased 3x3 convolutions with ReLU in five groups (2,2,3,3,3 of them for the
// 16-layer net, 2,2,4,4,4 for the 19-layer one), a 2x2/2 max pool after each
// group, three fully connected layers.  No batch norm, no dropout.
static void build_vgg16(const edl_config& c, Graph& g) {
    const int H = pick(c.H, 224), W = pick(c.W, 224), C = pick(c.C, 3), classes = pick(c.classes, 1000);
    const int base = pick(c.arch[0], 64), fc = pick(c.arch[1], 4096);
    int reps[5] = {2, 2, 3, 3, 3};
    if (c.arch[2] > 0) for (int i = 0; i < 5; ++i) reps[i] = c.arch[2 + i];
    const int mult[5] = {1, 2, 4, 8, 8};
    int t = g.add_tensor(H, W, C);
    int i = 0;
    char nm[16];
    for (int grp = 0; grp < 5; ++grp) {
        for (int r = 0; r < reps[grp]; ++r) {
            snprintf(nm, sizeof(nm), "conv%d", ++i);
            t = g.conv(t, base * mult[grp], 3, 1, 1, true, true, nm);
        }
        t = g.maxpool(t, 2, 2, 0);
    }
    t = g.flatten(t);
    t = g.conv(t, fc, 1, 1, 0, true, true, "fc1");
    t = g.conv(t, fc, 1, 1, 0, true, true, "fc2");
    t = g.conv(t, classes, 1, 1, 0, true, false, "fc3");
    g.loss(t);
}

// Five biased convolutions with ReLU (11x11/4 pad 2, 5x5 pad 2, three 3x3
// pad 1; base x {1,3,6,4,4} channels), a 3x3/2 max pool after the first, the
// second and the fifth, three fully connected layers.  The single-tower form
// without response normalisation; no dropout.
static void build_alexnet(const edl_config& c, Graph& g) {
    const int H = pick(c.H, 224), W = pick(c.W, 224), C = pick(c.C, 3), classes = pick(c.classes, 1000);
    const int base = pick(c.arch[0], 64), fc = pick(c.arch[1], 4096);
    int t = g.add_tensor(H, W, C);
    t = g.conv(t, base, 11, 4, 2, true, true, "conv1");
    t = g.maxpool(t, 3, 2, 0);
    t = g.conv(t, 3 * base, 5, 1, 2, true, true, "conv2");
    t = g.maxpool(t, 3, 2, 0);
    t = g.conv(t, 6 * base, 3, 1, 1, true, true, "conv3");
    t = g.conv(t, 4 * base, 3, 1, 1, true, true, "conv4");
    t = g.conv(t, 4 * base, 3, 1, 1, true, true, "conv5");
    t = g.maxpool(t, 3, 2, 0);
    t = g.flatten(t);
    t = g.conv(t, fc, 1, 1, 0, true, true, "fc1");
    t = g.conv(t, fc, 1, 1, 0, true, true, "fc2");
    t = g.conv(t, classes, 1, 1, 0, true, false, "fc3");
    g.loss(t);
}

int build_graph(const edl_config& cfg, Graph& g) {
    g = Graph();
    switch (cfg.model) {
        case EDL_MODEL_MLP: build_mlp(cfg, g); break;
        case EDL_MODEL_RESNET20: build_resnet20(cfg, g); break;
        case EDL_MODEL_RESNET50: build_resnet50(cfg, g); break;
        case EDL_MODEL_VGG16: build_vgg16(cfg, g); break;
        case EDL_MODEL_ALEXNET: build_alexnet(cfg, g); break;
        default: set_error("unknown model %d", cfg.model); return EDL_EINVAL;
    }
    for (const Tensor& t : g.tensors)
        if (t.H <= 0 || t.W <= 0 || t.C <= 0) {
            set_error("input image too small for this model");
            return EDL_EINVAL;
        }
    return EDL_OK;
}

}  // namespace edl

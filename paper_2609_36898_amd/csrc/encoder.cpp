// Host-side CSGV encoder (the preprocessing step: the paper compresses on the
// CPU, in parallel over bricks -- Methods > "Compressed segmentation volumes").
//
// Per brick: the finest level is the brick in Morton order; every coarser
// node is the mode of its 8 children (ties to the smaller label) and is
// flagged constant when its whole footprint holds one label.  Nodes are then
// visited coarse to fine in Morton order; a node is explicit when it is the
// root or its parent is explicit and not constant.  Each explicit node emits
// one operation -- the first applicable of PARENT, NX, NY, NZ, LAST, DELTA
// (unlimited delta, 4-bit entries, most significant group first), ADV --
// followed by the stop bit (= constant footprint; 0 on the finest level)
// (Results > "CSGV"; supplementary operation list).  The symbol streams of all
// bricks give one 16-symbol frequency table; each brick is stored with the
// plain 4-bit coder or interleaved rANS, whichever is smaller.
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <thread>
#include <vector>

#include "../../include/csgv.h"
#include "csgv_format.h"

using namespace csgv;

namespace {

struct Spread {
    uint32_t t[64];
    Spread() {
        for (uint32_t v = 0; v < 64; ++v) {
            uint32_t r = 0;
            for (int k = 0; k < 6; ++k) r |= ((v >> k) & 1u) << (3 * k);
            t[v] = r;
        }
    }
};
const Spread kSpread;

// byte c of t[m]: bit c of m
struct Bytes {
    uint64_t t[256];
    Bytes() {
        for (uint32_t m = 0; m < 256; ++m) {
            t[m] = 0;
            for (int c = 0; c < 8; ++c) t[m] |= (uint64_t)((m >> c) & 1u) << (8 * c);
        }
    }
};
const Bytes kBytes;
static_assert(kParent == 0 && kNX == 1 && kNY == 2 && kNZ == 3, "copies are coded as two bits");

// mode of 8 labels, ties to the smaller label (counted by all pairs: compares
// the compiler vectorises, where sorting them took three times as long)
template <typename LT>
inline LT mode_of8(const LT* c) {
    LT n[8];
    for (int i = 0; i < 8; ++i) n[i] = 0;
    for (int j = 0; j < 8; ++j)
        for (int i = 0; i < 8; ++i) n[i] += c[i] == c[j] ? 1 : 0;
    LT best = c[0], best_n = n[0];
    for (int i = 1; i < 8; ++i) {
        const bool take = n[i] > best_n || (n[i] == best_n && c[i] < best);
        best = take ? c[i] : best;
        best_n = take ? n[i] : best_n;
    }
    return best;
}

template <typename LT>
inline bool all_same(const LT* c) {
    LT d = 0;
    for (int j = 1; j < 8; ++j) d |= c[j] ^ c[0];
    return d == 0;
}

// label -> latest palette position, cleared in O(1) with a generation stamp.
// It grows with the palette (a brick has tens of labels as a rule, up to as many
// as nodes).
struct PosTable {
    std::vector<uint64_t> key;
    std::vector<uint32_t> val, gen;
    uint32_t mask = 0, cur = 0, used = 0;
    void reset() {
        if (key.empty()) resize(1024);
        used = 0;
        if (++cur == 0) {
            std::fill(gen.begin(), gen.end(), 0);
            cur = 1;
        }
    }
    void resize(size_t cap) {
        key.assign(cap, 0);
        val.assign(cap, 0);
        gen.assign(cap, 0);
        mask = (uint32_t)(cap - 1);
        cur = 0;
    }
    uint32_t slot(uint64_t k) const {
        uint32_t i = (uint32_t)((k * 0xD6E8FEB86659FD93ull) >> 40) & mask;
        while (gen[i] == cur && key[i] != k) i = (i + 1) & mask;
        return i;
    }
    bool find(uint64_t k, uint32_t* v) const {
        uint32_t i = slot(k);
        if (gen[i] != cur) return false;
        *v = val[i];
        return true;
    }
    void put(uint64_t k, uint32_t v) {
        if (2u * used > mask) {
            const std::vector<uint64_t> k0(std::move(key));
            const std::vector<uint32_t> v0(std::move(val)), g0(std::move(gen));
            const uint32_t c0 = cur;
            resize(2 * k0.size());
            cur = 1;
            for (size_t i = 0; i < k0.size(); ++i)
                if (g0[i] == c0) set(slot(k0[i]), k0[i], v0[i]);
        }
        const uint32_t i = slot(k);
        used += gen[i] != cur;
        set(i, k, v);
    }
    void set(uint32_t i, uint64_t k, uint32_t v) {
        gen[i] = cur;
        key[i] = k;
        val[i] = v;
    }
};

struct BrickCode {
    std::vector<uint8_t> sym;
    std::vector<uint64_t> pal;
    uint32_t sym_end[kMaxLog2b + 1] = {};
    uint32_t count[16] = {};  // of each symbol
    uint32_t L = 0;
    // chosen record
    std::vector<uint8_t> rec;
};

struct Worker {
    std::vector<uint64_t> lev[kMaxLog2b + 1];  // labels of a level, 4 or 8 bytes each
    std::vector<uint8_t> cst[kMaxLog2b + 1];
    std::vector<uint32_t> open, next;  // nodes whose children are explicit
    std::vector<uint8_t> sym;
    PosTable pos;
};

constexpr uint32_t kLegacyDelta = 16;  // longest palette back reference with op_mask bit 6

// A brick's operations.  The work is in its finest level: its nodes are put in
// Morton order, compared and reduced by whole 2x2x2 blocks, in the labels' own
// type, and a block that equals its parent is emitted at once.  (256^3 neurites, records
// included: 7.7 ms on a 16-core share with 64-bit labels, a flag per node, a
// sort per mixed block, a division per rANS symbol and the symbols counted by one
// thread, 2.5 now; on one core 101 ms and 57.)
template <typename LT>
void encode_brick(const uint8_t* vox, uint32_t L, uint32_t op_mask, uint32_t nmode, Worker& w, BrickCode& out) {
    const uint32_t b = 1u << L;
    LT* lev[kMaxLog2b + 1];
    for (uint32_t i = 0; i <= L; ++i) {
        const size_t n = size_t(1) << (3 * i);
        if (w.lev[i].size() < n) w.lev[i].resize(n);
        if (w.cst[i].size() < n) w.cst[i].resize(n);
        lev[i] = (LT*)w.lev[i].data();
    }
    // finest level, and the one above it
    {
        LT* const fine = lev[L];
        LT* const up = lev[L - 1];
        uint8_t* const uc = w.cst[L - 1].data();
        const uint32_t h = b / 2;
        for (uint32_t z = 0; z < h; ++z)
            for (uint32_t y = 0; y < h; ++y) {
                const uint32_t qyz = (kSpread.t[y] << 1) | (kSpread.t[z] << 2);
                const uint8_t* const row = vox + sizeof(LT) * (((size_t)2 * z * b + 2 * y) * b);
                for (uint32_t x = 0; x < h; ++x) {
                    const uint32_t q = kSpread.t[x] | qyz;
                    LT* const ch = fine + 8 * (size_t)q;
                    const uint8_t* const at = row + sizeof(LT) * 2 * x;
                    memcpy(ch, at, 2 * sizeof(LT));
                    memcpy(ch + 2, at + sizeof(LT) * b, 2 * sizeof(LT));
                    memcpy(ch + 4, at + sizeof(LT) * (size_t)b * b, 2 * sizeof(LT));
                    memcpy(ch + 6, at + sizeof(LT) * ((size_t)b * b + b), 2 * sizeof(LT));
                    const bool same = all_same(ch);
                    uc[q] = same;
                    up[q] = same ? ch[0] : mode_of8(ch);
                }
            }
    }
    for (uint32_t i = L - 1; i >= 1; --i) {
        const size_t np = size_t(1) << (3 * (i - 1));
        for (size_t q = 0; q < np; ++q) {
            const LT* const ch = lev[i] + 8 * q;
            uint64_t cc;
            memcpy(&cc, w.cst[i].data() + 8 * q, 8);
            const bool same = all_same(ch);
            w.cst[i - 1][q] = same && cc == 0x0101010101010101ull;
            lev[i - 1][q] = same ? ch[0] : mode_of8(ch);
        }
    }
    // traversal
    out.L = L;
    out.pal.clear();
    w.pos.reset();
    constexpr size_t kMost = 8 * 12 + 8;  // symbols of 8 nodes, an operation and up to 11 entries each, and a whole store
    if (w.sym.size() < 4096) w.sym.resize(4096);
    uint8_t* sym = w.sym.data();
    size_t ns = 0;
    // a node that neither its parent nor a neighbour names: LAST, DELTA or ADV
    const auto palette_op = [&](LT v, uint32_t stop) {
        uint32_t op = kAdv, delta = 0, p;
        if ((op_mask & 16u) && !out.pal.empty() && out.pal.back() == v) op = kLast;
        // bit 6: back references of at most kLegacyDelta entries, as in the original
        // format; a label further back is appended again (a palette duplicate)
        else if ((op_mask & 32u) && w.pos.find(v, &p) && (!(op_mask & 64u) || out.pal.size() - p <= kLegacyDelta)) {
            op = kDelta;
            delta = (uint32_t)out.pal.size() - p;
        }
        if (op == kAdv) {
            if (op_mask & 32u) w.pos.put(v, (uint32_t)out.pal.size());  // (read by back references only)
            out.pal.push_back(v);
        }
        sym[ns++] = (uint8_t)(op | (stop << 3));
        if (op == kDelta) {
            int groups = 1;
            while (groups < 11 && (delta >> (3 * groups)) != 0) ++groups;
            for (int g = groups - 1; g >= 0; --g) sym[ns++] = (uint8_t)(((delta >> (3 * g)) & 7u) | (g > 0 ? 8u : 0u));
        }
    };
    // children of a block that may copy from their neighbour along an axis: in
    // neighbour mode 1 only from another sibling group (an even coordinate)
    const uint32_t inner = nmode ? 0u : 0xFFu;
    const uint32_t from[3] = {op_mask & 2u ? 0x55u | (inner & 0xAAu) : 0u, op_mask & 4u ? 0x33u | (inner & 0xCCu) : 0u,
                              op_mask & 8u ? 0x0Fu | (inner & 0xF0u) : 0u};
    palette_op(lev[0][0], w.cst[0][0]);
    out.sym_end[0] = (uint32_t)ns;
    w.open.assign(1, 0);
    size_t n_open = w.cst[0][0] ? 0 : 1;
    for (uint32_t i = 1; i <= L; ++i) {
        const uint32_t mx = 0x09249249u & ((1u << (3 * (i - 1))) - 1u);  // of the blocks' nodes
        const LT* const cur = lev[i];
        const uint8_t* const cst = w.cst[i].data();
        if (i < L && w.next.size() < 8 * n_open) w.next.resize(8 * n_open);
        size_t n_next = 0;
        for (size_t k = 0; k < n_open; ++k) {
            const uint32_t q = w.open[k];
            if (ns + kMost > w.sym.size()) {
                w.sym.resize(2 * w.sym.size());
                sym = w.sym.data();
            }
            const LT* const ch = cur + 8 * (size_t)q;
            const LT pv = lev[i - 1][q];
            uint32_t same[3] = {0, 0, 0}, par = 0, stop = 0;
            for (uint32_t c = 0; c < 8; ++c) par |= (uint32_t)(ch[c] == pv) << c;
            if (!(op_mask & 1u)) par = 0;
            if (par != 0xFFu) {
                // the neighbours: siblings, or the facing children of the block before
                // this one along the axis (of this block itself, masked, at the border)
                for (uint32_t a = 0; a < 3; ++a) {
                    const uint32_t bit = 1u << a, am = mx << a;
                    const LT* const nb = q & am ? cur + 8 * (size_t)((((q & am) - 1u) & am) | (q & ~am)) : ch;
                    for (uint32_t c = 0; c < 8; ++c) same[a] |= (uint32_t)(ch[c] == (c & bit ? ch[c ^ bit] : nb[c | bit])) << c;
                    same[a] &= q & am ? from[a] : from[a] & (a == 0 ? 0xAAu : a == 1 ? 0xCCu : 0xF0u);
                }
            }
            if (i < L)
                for (uint32_t c = 0; c < 8; ++c) {
                    const uint32_t st = cst[8 * (size_t)q + c];
                    stop |= st << c;
                    w.next[n_next] = 8 * q + c;
                    n_next += 1u - st;
                }
            const uint32_t x = same[0] & ~par, y = same[1] & ~(par | x), z = same[2] & ~(par | x | y);
            uint64_t all = kBytes.t[x | z] | (kBytes.t[y | z] << 1) | (kBytes.t[stop] << 3);
            uint32_t pos = 0;
            for (uint32_t rest = 0xFFu & ~(par | x | y | z); rest; rest &= rest - 1u) {
                const uint32_t c = (uint32_t)__builtin_ctz(rest);
                memcpy(sym + ns, &all, 8);
                ns += c - pos;
                palette_op(ch[c], (stop >> c) & 1u);
                all = c < 7 ? all >> (8 * (c + 1 - pos)) : 0;
                pos = c + 1;
            }
            memcpy(sym + ns, &all, 8);
            ns += 8 - pos;
        }
        out.sym_end[i] = (uint32_t)ns;
        std::swap(w.open, w.next);
        n_open = n_next;
    }
    out.sym.assign(sym, sym + ns);
    uint32_t cnt[4][16] = {};  // (four tables: a run of one symbol does not wait for its own count)
    for (size_t k = 0; k < ns; ++k) ++cnt[k & 3][sym[k]];
    for (int v = 0; v < 16; ++v) out.count[v] = cnt[0][v] + cnt[1][v] + cnt[2][v] + cnt[3][v];
}

// normalised table (sum 4096): floor(count * 4096 / total), at least 1 for
// used symbols; shortfall to the most frequent symbol (lowest on ties); any
// excess taken one by one from the largest entry above 1 (lowest on ties)
void normalise(const uint64_t cnt[16], uint16_t f[16]) {
    uint64_t tot = 0;
    for (int s = 0; s < 16; ++s) tot += cnt[s];
    if (!tot) {
        memset(f, 0, 32);
        return;
    }
    int64_t sum = 0;
    for (int s = 0; s < 16; ++s) {
        uint64_t v = cnt[s] ? std::max<uint64_t>(1, cnt[s] * kRansM / tot) : 0;
        f[s] = (uint16_t)v;
        sum += (int64_t)v;
    }
    if (sum < (int64_t)kRansM) {
        int best = 0;
        for (int s = 1; s < 16; ++s)
            if (cnt[s] > cnt[best]) best = s;
        f[best] = (uint16_t)(f[best] + (kRansM - sum));
    }
    while (sum > (int64_t)kRansM) {
        int best = -1;
        for (int s = 0; s < 16; ++s)
            if (f[s] > 1 && (best < 0 || f[s] > f[best])) best = s;
        --f[best];
        --sum;
    }
}

inline void put32(std::vector<uint8_t>& v, size_t at, uint32_t x) { memcpy(&v[at], &x, 4); }

// The rANS step of one symbol, x -> (x / f) * 4096 + x % f + cum, as a
// multiplication: q = x * rcp >> 64 is x / f for x < 2^32 and f <= 4096 (Granlund
// and Montgomery, "Division by invariant integers using multiplication", 1994),
// and the step is x + bias + q * (4096 - f).  f = 1 has no 64-bit reciprocal:
// its q is x - 1, which its bias makes good.  (The four quantities per symbol and
// the way out for f = 1 are those of Giesen's public-domain rANS coder, 2014.)
struct RansStep {
    uint64_t rcp, limit;
    uint32_t bias, rest;
};

void rans_steps(const uint16_t* freq, const uint32_t* cum, RansStep st[16]) {
    for (int s = 0; s < 16; ++s) {
        const uint32_t f = freq[s];
        st[s].limit = (uint64_t)f << 20;
        st[s].rcp = f > 1 ? ~0ull / f + 1u : ~0ull;
        st[s].bias = cum[s] + (f > 1 ? 0u : kRansM - 1u);
        st[s].rest = kRansM - f;
    }
}

// A brick's record, with the plain 4-bit coder (policy 1), interleaved rANS (2),
// or whichever is smaller, the plain one on ties (0: its size is known without
// building it).
void build_record(BrickCode& bc, uint32_t lb, uint32_t policy, uint32_t lane_syms, const RansStep* steps,
                  std::vector<uint16_t>& words) {
    const uint32_t L = bc.L, nsym = (uint32_t)bc.sym.size(), pc = (uint32_t)bc.pal.size();
    const size_t al = lb == 8 ? 8 : 4;
    const auto palette_at = [&](uint32_t coder, uint32_t log2W) {
        return (record_header_bytes(L, coder, log2W) + al - 1) / al * al;
    };
    const auto bytes = [&](size_t pal_off, size_t pay) { return (pal_off + (size_t)pc * lb + pay + 7) / 8 * 8; };
    uint32_t log2W = 0, W = 1, G = 1, state[256], begin[5] = {0, 0, 0, 0, 0}, at[4] = {0, 0, 0, 0};
    size_t pay = (nsym + 1) / 2, total = bytes(palette_at(kRaw4, 0), pay);
    bool rans = false;
    if (policy != 1) {
        while (W < 256 && (uint64_t)W * 2 * lane_syms <= nsym) {
            W *= 2;
            ++log2W;
        }
        G = (W + 63) / 64;
        // every lane group's words, backwards from the end of its share: a symbol emits one at most
        for (uint32_t g = 0; g < G; ++g) begin[g + 1] = begin[g] + std::min(W, 64u) * (nsym / W + 1);
        if (words.size() < begin[G]) words.resize(begin[G]);
        for (uint32_t g = 0; g < G; ++g) at[g] = begin[g + 1];
        for (uint32_t l = 0; l < W; ++l) state[l] = kRansL;
        const uint8_t* const sym = bc.sym.data();
        // (whole rounds group by group: the stores' place stays in a register)
        for (uint32_t g = 0; g < G; ++g) {
            const uint32_t lanes = W < 64 ? W : 64;
            uint16_t* out = words.data() + at[g];
            uint32_t* const sg = state + 64 * g;
            for (uint32_t r = (nsym + W - 1) / W; r-- > 0;) {
                const uint32_t j0 = r * W + 64 * g, n = j0 >= nsym ? 0u : std::min(lanes, nsym - j0);
                for (uint32_t l = n; l-- > 0;) {
                    const RansStep& st = steps[sym[j0 + l]];
                    uint32_t x = sg[l];
                    out[-1] = (uint16_t)x;
                    const bool full = x >= st.limit;
                    out -= full;
                    x = full ? x >> 16 : x;
                    const uint32_t q = (uint32_t)(((unsigned __int128)x * st.rcp) >> 64);
                    sg[l] = x + st.bias + q * st.rest;
                }
            }
            at[g] = (uint32_t)(out - words.data());
        }
        size_t rpay = 0;
        for (uint32_t g = 0; g < G; ++g) rpay += 2 * (size_t)(begin[g + 1] - at[g]);
        const size_t rtotal = bytes(palette_at(kRans, log2W), rpay);
        rans = policy == 2 || rtotal < total;
        if (rans) {
            pay = rpay;
            total = rtotal;
        }
    }
    if (!rans) log2W = 0, W = G = 1;
    const size_t pal_off = palette_at(rans ? kRans : kRaw4, log2W), pay_off = pal_off + (size_t)pc * lb;
    std::vector<uint8_t>& rec = bc.rec;
    rec.assign(total, 0);
    rec[0] = (uint8_t)(rans ? kRans : kRaw4);
    rec[1] = (uint8_t)L;
    rec[2] = (uint8_t)lb;
    rec[3] = (uint8_t)log2W;
    put32(rec, 4, pc);
    for (uint32_t i = 0; i <= L; ++i) put32(rec, 8 + 4 * i, bc.sym_end[i]);
    if (rans) {
        size_t o = 8 + 4 * (L + 1);
        for (uint32_t g = 0; g < G; ++g) put32(rec, o + 4 * g, begin[g + 1] - at[g]);
        o += 4 * G;
        memcpy(&rec[o], state, 4 * (size_t)W);
    }
    for (uint32_t k = 0; k < pc; ++k) {
        if (lb == 8) memcpy(&rec[pal_off + 8 * (size_t)k], &bc.pal[k], 8);
        else {
            uint32_t v = (uint32_t)bc.pal[k];
            memcpy(&rec[pal_off + 4 * (size_t)k], &v, 4);
        }
    }
    if (!rans) {
        for (uint32_t j = 0; j < nsym; ++j) rec[pay_off + j / 2] |= (uint8_t)(bc.sym[j] << (4 * (j & 1)));
    } else {
        size_t o = pay_off;
        for (uint32_t g = 0; g < G; ++g) {
            const size_t n = 2 * (size_t)(begin[g + 1] - at[g]);
            if (n) memcpy(&rec[o], &words[at[g]], n);
            o += n;
        }
    }
}

// Threads worth starting for n items of `ns` nanoseconds of work in all, the calling
// one included: one per 200 us, twice what starting and joining it costs (40 us of
// the starting thread and a wake-up; 7 threads and no work: 0.35 ms).
constexpr double kThreadNs = 2e5;
int threads_for(int threads, uint32_t n, double ns) {
    return (int)std::max(1.0, std::min({(double)threads, (double)n, ns / kThreadNs}));
}

// About the nanoseconds that a brick's operations take: 4 a voxel, and 30 more for one that
// can copy from no neighbour, judged by how often voxels of four of the brick's rows differ
// from the one before them, for two axes (smooth labels 3 to 5 ns a voxel, 16 labels at
// random 29, noise 32 to 42 and at side 64, where its label table leaves the caches, 105).
// The number of bricks says little: 4 of 64^3 with 16 random labels take 37 ms with one
// thread and 16 with four, 4 smooth ones of 16^3 take 0.12 with one and 1.4 with eight.
template <typename LT>
double brick_ns(const uint8_t* vox, uint32_t L) {
    const uint32_t b = 1u << L;
    uint32_t seen = 0, differ = 0;
    for (uint32_t r = 0; r < 4; ++r) {
        const uint32_t y = (2u * r + 1u) * b / 8u, z = (2u * (r ^ 1u) + 1u) * b / 8u;
        const uint8_t* const row = vox + sizeof(LT) * (((size_t)z * b + y) * b);
        LT last, v;
        memcpy(&last, row, sizeof(LT));
        for (uint32_t x = 1; x < b; ++x, last = v) {
            memcpy(&v, row + sizeof(LT) * x, sizeof(LT));
            ++seen;
            differ += v != last;
        }
    }
    const double f = (double)differ / seen;
    return (double)(size_t(1) << (3 * L)) * (4.0 + 30.0 * f * f);
}

// fn(item, thread) for every item on `threads` threads, the calling one among them
template <class F>
void parallel_for(uint32_t n, int threads, F&& fn) {
    std::atomic<uint32_t> next{0};
    const auto work = [&](int t) {
        for (;;) {
            const uint32_t i = next.fetch_add(1);
            if (i >= n) break;
            fn(i, t);
        }
    };
    std::vector<std::thread> pool;
    for (int t = 1; t < threads; ++t) pool.emplace_back(work, t);
    work(0);
    for (auto& th : pool) th.join();
}

}  // namespace

// Streaming encoder: bricks are symbolised as they are added (the raw voxels
// can be dropped right after), the volume's frequency table and the records
// are produced once at the end.
struct csgv_encoder {
    uint32_t label_bytes = 4, default_log2b = 5, op_mask = 63, neighbor_mode = 0, coder_policy = 0, lane_syms = 64;
    uint32_t dims[3] = {0, 0, 0}, grid[3] = {0, 0, 0};
    bool has_grid = false, with_dir = false;
    int threads = 1;
    std::vector<BrickCode> bc;
    std::vector<uint32_t> origins;  // 3 per brick when with_dir
    std::vector<uint8_t> log2b;
};

extern "C" {

csgv_status csgv_encoder_create(uint32_t label_bytes, const uint32_t dims[3], uint32_t default_log2b,
                                const uint32_t grid[3], int with_directory, uint32_t op_mask, uint32_t neighbor_mode,
                                uint32_t coder_policy, uint32_t lane_syms, int n_threads, csgv_encoder** out) {
    if (!out) return CSGV_EINVAL;
    if (label_bytes != 4 && label_bytes != 8) return CSGV_EINVAL;
    if (coder_policy > 2) return CSGV_EINVAL;
    csgv_encoder* e = new csgv_encoder();
    e->label_bytes = label_bytes;
    e->default_log2b = default_log2b;
    e->op_mask = op_mask;
    e->neighbor_mode = neighbor_mode;
    e->coder_policy = coder_policy;
    e->lane_syms = lane_syms < 1 ? 1 : lane_syms;
    for (int a = 0; a < 3; ++a) {
        e->dims[a] = dims ? dims[a] : 0;
        e->grid[a] = grid ? grid[a] : 0;
    }
    e->with_dir = with_directory != 0;
    e->threads = n_threads > 0 ? n_threads : (int)std::max(1u, std::thread::hardware_concurrency());
    *out = e;
    return CSGV_OK;
}

csgv_status csgv_encoder_add(csgv_encoder* e, const void* h_voxels, const uint8_t* h_log2b, uint32_t n_bricks,
                             const uint32_t* h_origins) {
    if (!e || (n_bricks && (!h_voxels || !h_log2b))) return CSGV_EINVAL;
    if (e->with_dir && n_bricks && !h_origins) return CSGV_EINVAL;
    std::vector<size_t> vox_off(n_bricks + 1, 0);
    for (uint32_t k = 0; k < n_bricks; ++k) {
        if (h_log2b[k] < 1 || h_log2b[k] > kMaxLog2b) return CSGV_EINVAL;
        vox_off[k + 1] = vox_off[k] + (size_t(1) << (3 * h_log2b[k]));
    }
    const size_t base = e->bc.size();
    e->bc.resize(base + n_bricks);
    const uint8_t* vox = (const uint8_t*)h_voxels;
    const uint32_t lb = e->label_bytes;
    double ns = 0;
    for (uint32_t k = 0; k < n_bricks && ns < kThreadNs * e->threads; ++k) {
        const uint8_t* const v = vox + vox_off[k] * lb;
        ns += lb == 4 ? brick_ns<uint32_t>(v, h_log2b[k]) : brick_ns<uint64_t>(v, h_log2b[k]);
    }
    const int threads = threads_for(e->threads, n_bricks, ns);
    std::vector<Worker> workers(threads);
    parallel_for(n_bricks, threads, [&](uint32_t k, int t) {
        const uint8_t* const v = vox + vox_off[k] * lb;
        if (lb == 4) encode_brick<uint32_t>(v, h_log2b[k], e->op_mask, e->neighbor_mode, workers[t], e->bc[base + k]);
        else encode_brick<uint64_t>(v, h_log2b[k], e->op_mask, e->neighbor_mode, workers[t], e->bc[base + k]);
    });
    e->log2b.insert(e->log2b.end(), h_log2b, h_log2b + n_bricks);
    if (e->with_dir) e->origins.insert(e->origins.end(), h_origins, h_origins + 3ull * n_bricks);
    return CSGV_OK;
}

csgv_status csgv_encoder_finish(csgv_encoder* e, void** h_out, uint64_t* out_bytes) {
    if (!e || !h_out || !out_bytes) return CSGV_EINVAL;
    const uint32_t n_bricks = (uint32_t)e->bc.size();
    const uint32_t label_bytes = e->label_bytes, lane_syms = e->lane_syms, coder_policy = e->coder_policy;
    std::vector<BrickCode>& bc = e->bc;
    uint64_t cnt[16] = {0};
    for (auto& c : bc)
        for (int s = 0; s < 16; ++s) cnt[s] += c.count[s];
    uint16_t freq[16];
    normalise(cnt, freq);
    uint32_t cum[17];
    cum[0] = 0;
    for (int s = 0; s < 16; ++s) cum[s + 1] = cum[s] + freq[s];
    RansStep steps[16];
    rans_steps(freq, cum, steps);
    // (2 to 5 ns a symbol with its palette entry)
    double ns = 0;
    for (auto& c : bc) ns += 2.0 * (double)(c.sym.size() + c.pal.size());
    const int threads = threads_for(e->threads, n_bricks, ns);
    std::vector<std::vector<uint16_t>> words(threads);
    parallel_for(n_bricks, threads, [&](uint32_t k, int t) {
        build_record(bc[k], label_bytes, coder_policy, lane_syms, steps, words[t]);
        std::vector<uint8_t>().swap(bc[k].sym);
        std::vector<uint64_t>().swap(bc[k].pal);
    });
    const bool dir = e->with_dir;
    const uint64_t off_pos = kHeaderBytes;
    const uint64_t dir_pos = dir ? (off_pos + 8ull * (n_bricks + 1) + 7) / 8 * 8 : 0;
    uint64_t rec0 = dir ? dir_pos + 16ull * n_bricks : off_pos + 8ull * (n_bricks + 1);
    rec0 = (rec0 + 7) / 8 * 8;
    uint64_t total = rec0;
    for (auto& c : bc) total += c.rec.size();
    uint8_t* buf = (uint8_t*)calloc(total ? total : 1, 1);
    if (!buf) return CSGV_ENOMEM;
    auto w32 = [&](uint64_t at, uint32_t v) { memcpy(buf + at, &v, 4); };
    auto w64 = [&](uint64_t at, uint64_t v) { memcpy(buf + at, &v, 8); };
    w32(0, kMagic);
    w32(4, kVersion);
    for (int a = 0; a < 3; ++a) {
        w32(kHdrDims + 4 * a, e->dims[a]);
        w32(kHdrGrid + 4 * a, e->grid[a]);
    }
    w32(kHdrLog2b, e->default_log2b);
    w32(kHdrLabelBytes, label_bytes);
    w32(kHdrOpMask, e->op_mask);
    w32(kHdrNBricks, n_bricks);
    memcpy(buf + kHdrFreq, freq, 32);
    w64(kHdrOffsetsPos, off_pos);
    w64(kHdrDirPos, dir_pos);
    w64(kHdrTotal, total);
    w32(kHdrNeighborMode, e->neighbor_mode);
    uint64_t pos = rec0;
    for (uint32_t k = 0; k < n_bricks; ++k) {
        w64(off_pos + 8ull * k, pos);
        if (dir) {
            for (int a = 0; a < 3; ++a) w32(dir_pos + 16ull * k + 4 * a, e->origins[3ull * k + a]);
            w32(dir_pos + 16ull * k + 12, e->log2b[k]);
        }
        pos += bc[k].rec.size();
    }
    w64(off_pos + 8ull * n_bricks, pos);
    // (0.25 ns a byte, most of it the fresh pages')
    parallel_for(n_bricks, threads_for(e->threads, n_bricks, 0.25 * (double)total), [&](uint32_t k, int) {
        uint64_t at;
        memcpy(&at, buf + off_pos + 8ull * k, 8);
        memcpy(buf + at, bc[k].rec.data(), bc[k].rec.size());
        std::vector<uint8_t>().swap(bc[k].rec);
    });
    bc.clear();
    *h_out = buf;
    *out_bytes = total;
    return CSGV_OK;
}

void csgv_encoder_destroy(csgv_encoder* e) { delete e; }

csgv_status csgv_encode_bricks(const void* h_voxels, const uint8_t* h_log2b, uint32_t n_bricks, uint32_t label_bytes,
                               const uint32_t dims[3], uint32_t default_log2b, const uint32_t grid[3],
                               const uint32_t* h_origins, uint32_t op_mask, uint32_t neighbor_mode,
                               uint32_t coder_policy, uint32_t lane_syms, int n_threads, void** h_out,
                               uint64_t* out_bytes) {
    if (!h_out || !out_bytes || (n_bricks && (!h_voxels || !h_log2b))) return CSGV_EINVAL;
    csgv_encoder* e = nullptr;
    csgv_status st = csgv_encoder_create(label_bytes, dims, default_log2b, grid, h_origins != nullptr, op_mask,
                                         neighbor_mode, coder_policy, lane_syms, n_threads, &e);
    if (st != CSGV_OK) return st;
    st = csgv_encoder_add(e, h_voxels, h_log2b, n_bricks, h_origins);
    if (st == CSGV_OK) st = csgv_encoder_finish(e, h_out, out_bytes);
    csgv_encoder_destroy(e);
    return st;
}

}  // extern "C"

// Trace loading: JSON-lines parser, array import, candidate-independent preprocessing.
//
// The replay input is a Mooncake-style trace (Sec. 3 "Dataset": per-request timestamps, request metadata,
// block hash ids).  Everything that does not depend on the candidate weights is done here once: hash ids
// are renumbered densely (1 + order of first appearance), repeated ids inside one request are flagged, and
// the trace is classified as chain-consistent or not.
#include <algorithm>
#include <cerrno>
#include <cstdio>
#include <cstring>
#include <cstdlib>
#include <limits>
#include <memory>
#include <new>
#include <string>
#include <sys/stat.h>
#include <thread>

#include "internal.h"

namespace gorgo {

static thread_local std::string g_err;

int fail(int code, const std::string& msg) {
    g_err = msg;
    return code;
}
void clear_error() { g_err.clear(); }

namespace {

// What preprocessing knows of a key (a distinct block id; keys are numbered from 1 in order of first appearance).
struct KeyInfo {
    int64_t id = 0;
    uint32_t parent = 0, pos = 0;    // predecessor and position it was first seen with
    uint32_t next = 0;               // key that followed it last
    uint32_t nchild = 0;             // distinct successors
    int32_t seen_in = -1;            // last request that it was seen in
    uint8_t ends = 0;                // some request ends here
};

// The block ids of a trace's requests, one after the other, as they lie in memory: in one array, or in several, each with the ids
// of whole requests from block `from` on.
struct IdRun {
    int64_t from;
    const int64_t* ids;
};
class Ids {
  public:
    explicit Ids(const std::vector<IdRun>& runs) : runs_(runs) {}
    // those of a request whose first block is b; called with increasing b
    const int64_t* of(int64_t b) {
        while (at_ + 1 < runs_.size() && runs_[at_ + 1].from <= b) ++at_;
        return runs_[at_].ids + (b - runs_[at_].from);
    }

  private:
    const std::vector<IdRun>& runs_;
    size_t at_ = 0;
};

// Open-addressed map from ids to keys: linear probing over the keys' numbers alone (0: empty), grows fourfold (by doubling, keys
// are entered twice as often again).
class IdMap {
  public:
    // (a table of half the trace's blocks, up to 4 MiB, to begin with: growing costs more than clearing it)
    IdMap(std::vector<KeyInfo>& keys, int64_t blocks) : keys_(keys) {
        size_t n = (size_t)1 << 12;
        while (n < ((size_t)1 << 20) && n < (size_t)blocks / 2) n *= 2;
        slot_.assign(n, 0);
    }
    // the key of an id, the next one on first sight
    uint32_t get_or_add(int64_t id, bool* added) {
        if (keys_.size() * 2 > slot_.size()) grow();
        size_t h = mix((uint64_t)id) & (slot_.size() - 1);
        while (slot_[h] != 0) {
            if (keys_[slot_[h]].id == id) { *added = false; return slot_[h]; }
            h = (h + 1) & (slot_.size() - 1);
        }
        slot_[h] = (uint32_t)keys_.size();
        keys_.emplace_back();
        keys_.back().id = id;
        *added = true;
        return slot_[h];
    }

  private:
    static uint64_t mix(uint64_t x) {
        x ^= x >> 30; x *= 0xbf58476d1ce4e5b9ULL;
        x ^= x >> 27; x *= 0x94d049bb133111ebULL;
        return x ^ (x >> 31);
    }
    void grow() {
        slot_.assign(slot_.size() * 4, 0);
        for (size_t k = 1; k < keys_.size(); ++k) {
            size_t h = mix((uint64_t)keys_[k].id) & (slot_.size() - 1);
            while (slot_[h] != 0) h = (h + 1) & (slot_.size() - 1);
            slot_[h] = (uint32_t)k;
        }
    }
    std::vector<KeyInfo>& keys_;
    std::vector<uint32_t> slot_;
};

// Row slots of single blocks, for traces that do not go by segments: an id has a slot from its first to its last request (see
// the segments' below; reused oldest-first, not before the next request).
int block_rows(gorgo_trace* t, const std::vector<KeyInfo>& keys) {
    const int64_t N = t->N, total = t->total_blocks;
    struct Use { int32_t last = -1, slot = -1, born = -1, seen = -2, before = -2; };      // `seen`: latest request so far
    std::vector<Use> use(keys.size());
    for (size_t k = 1; k < keys.size(); ++k) use[k].last = keys[k].seen_in;
    std::vector<int32_t> free_slots, gone;
    size_t head = 0;
    int32_t n_slots = 0;
    t->row_ref.resize((size_t)total);
    for (int64_t r = 0; r < N; ++r) {
        for (int64_t j = t->blk_off[r]; j < t->blk_off[r + 1]; ++j) {
            Use& of = use[t->key[(size_t)j]];
            if (of.slot < 0) {
                if (head >= free_slots.size() && (uint32_t)n_slots >= ROW_SLOT) {        // (too many: tables only)
                    t->row_ref.clear();
                    return GORGO_OK;
                }
                of.slot = head < free_slots.size() ? free_slots[head++] : n_slots++;
                of.born = (int32_t)r;
            }
            if (of.seen != r) {
                of.before = of.seen;
                of.seen = (int32_t)r;
            }
            const bool first = t->first[(size_t)j] != 0;
            t->row_ref[(size_t)j] = (uint32_t)of.slot | (first ? ROW_FIRST : 0u) | (of.before == r - 1 ? ROW_IN_BEFORE : 0u) |
                                    (of.born == r ? ROW_FRESH : of.born == r - 1 ? ROW_NEW_BEFORE : 0u);
            if (first && of.last == r) gone.push_back(of.slot);
        }
        free_slots.insert(free_slots.end(), gone.begin(), gone.end());
        gone.clear();
    }
    t->n_row_slots = n_slots;
    return GORGO_OK;
}

// Fills key/first/statistics from the raw ids.  Returns 0 or an error code.
int preprocess(gorgo_trace* t, const std::vector<IdRun>& runs) {
    const int64_t N = t->N;
    const int64_t total = t->blk_off[N];
    t->total_blocks = total;
    t->key.resize((size_t)total);
    t->first.resize((size_t)total);
    std::vector<KeyInfo> keys;
    keys.reserve((size_t)std::min<int64_t>(total, 1 << 20) + 1);
    keys.emplace_back();             // (key 0 stands before a request's first block)
    IdMap map(keys, total);
    Ids ids(runs);
    bool consistent = true;
    int32_t max_blocks = 0, max_distinct = 0;
    uint32_t* const out = t->key.data();       // (by value: a byte that is written may be anything, also where a vector lies)
    uint8_t* const first = t->first.data();
    KeyInfo* info = keys.data();
    for (int64_t r = 0; r < N; ++r) {
        const int64_t b = t->blk_off[r], e = t->blk_off[r + 1];
        const int64_t n = e - b;
        if (n > max_blocks) max_blocks = (int32_t)n;
        int32_t distinct = 0;
        uint32_t prev = 0;
        size_t known = keys.size();
        const int64_t* const its = n > 0 ? ids.of(b) : nullptr;
        for (int64_t k = 0; k < n; ++k) {
            // Prompts repeat each other's beginnings: an id is mostly the one that first appeared behind its predecessor, or else
            // the one that followed it the last time, and needs no look-up.
            const int64_t id = its[k];
            bool added = false;
            uint32_t key = prev + 1;
            if (prev == 0 || key >= known || info[key].id != id) {
                key = prev ? info[prev].next : 0;
                if (key == 0 || info[key].id != id) {
                    key = map.get_or_add(id, &added);
                    known = keys.size();
                    info = keys.data();
                    if (known > 0xFFFFFFF0ull) return fail(GORGO_ERR_INVALID_ARG, "too many distinct hash ids");
                    if (prev) info[prev].next = key;
                }
            }
            KeyInfo& of = info[key];
            if (added) {
                of.parent = prev;
                of.pos = (uint32_t)k;
                if (prev) ++info[prev].nchild;
            } else if (of.parent != prev || of.pos != (uint32_t)k) {
                consistent = false;
            }
            const bool dup = of.seen_in == (int32_t)r;
            if (dup) consistent = false;
            else ++distinct;
            of.seen_in = (int32_t)r;
            out[b + k] = key;
            first[b + k] = dup ? 0 : 1;
            prev = key;
        }
        if (prev) info[prev].ends = 1;
        if (distinct > max_distinct) max_distinct = distinct;
    }
    t->max_blocks = max_blocks;
    t->max_distinct = max_distinct;
    t->unique_ids = (int64_t)keys.size() - 1;
    t->chain_consistent = consistent;
    t->seg_off.clear();
    t->seg.clear();
    t->n_segments = 0;
    t->n_slots = 0;
    t->seg_prev.clear();
    t->row_ref.clear();
    t->n_row_slots = 0;
    if (!consistent) return block_rows(t, keys);

    // Chain-consistent traces: the keys form a forest and every request is a root-to-node path.  Cut the
    // forest into segments -- maximal runs of keys with a single successor and no request ending inside --
    // so that every request is a whole number of segments and all blocks of a segment are always touched
    // together.  Keys are numbered in order of first appearance, so a predecessor precedes its successors.
    const size_t U = keys.size() - 1;
    std::vector<int32_t> seg_of(U + 1, 0);
    std::vector<int32_t> seg_end;          // of each segment: blocks of a request up to and including it
    int64_t nseg = 0;
    for (size_t k = 1; k <= U; ++k) {
        const uint32_t par = keys[k].parent;
        if (par == 0 || keys[par].nchild > 1 || keys[par].ends) {
            seg_of[k] = (int32_t)(nseg++);
            seg_end.push_back(0);
        } else {
            seg_of[k] = seg_of[par];
        }
        seg_end[(size_t)seg_of[k]] = (int32_t)keys[k].pos + 1;       // (its last key has the highest number)
        if (nseg >= 0x7FFFFFF0) return fail(GORGO_ERR_INVALID_ARG, "too many segments");
    }
    t->n_segments = nseg;
    t->seg_off.resize((size_t)N + 1);
    t->seg_off[0] = 0;
    for (int64_t r = 0; r < N; ++r) {
        const int64_t b = t->blk_off[r], e = t->blk_off[r + 1];
        for (int64_t k = b; k < e; k = b + t->seg.back().end) {      // (whole segments)
            const int32_t sg = seg_of[t->key[(size_t)k]];
            t->seg.push_back(gorgo::SegRef{sg, seg_end[(size_t)sg]});
        }
        t->seg_off[(size_t)r + 1] = (int64_t)t->seg.size();
    }

    // Row slots.  The replay keeps one row of cells per segment, but a segment only matters between the first and
    // the last request that reference it (no candidate can change that: it is a property of the trace), and at any
    // time only the segments of conversations still going on are between the two.  So segments share rows: a
    // segment takes a slot at its first reference -- marked SEG_FRESH in that reference, where the replay resets
    // the row before anything reads it -- and gives it back after its last one.  Slots are reused oldest-first.
    std::vector<int32_t> last_ref((size_t)nseg, -1);
    t->seg_prev.resize(t->seg.size());
    for (int64_t r = 0; r < N; ++r)
        for (int64_t j = t->seg_off[(size_t)r]; j < t->seg_off[(size_t)r + 1]; ++j) {
            int32_t& of = last_ref[(size_t)t->seg[(size_t)j].id];
            t->seg_prev[(size_t)j] = of;
            of = (int32_t)r;
        }
    std::vector<int32_t> slot_of((size_t)nseg, -1);
    std::vector<int32_t> free_slots;       // a queue: taken from `head`, given back at the end
    size_t head = 0;
    int32_t n_slots = 0;
    std::vector<int32_t> seg_at;           // segments of the request in hand, by place in its path
    for (int64_t r = 0; r < N; ++r) {
        const int64_t j0 = t->seg_off[(size_t)r], j1 = t->seg_off[(size_t)r + 1];
        seg_at.clear();
        for (int64_t j = j0; j < j1; ++j) {
            gorgo::SegRef& ref = t->seg[(size_t)j];
            const size_t sg = (size_t)ref.id;
            seg_at.push_back(ref.id);
            if (slot_of[sg] < 0) {
                slot_of[sg] = head < free_slots.size() ? free_slots[head++] : n_slots++;
                ref.end |= gorgo::SEG_FRESH;
            }
            ref.id = slot_of[sg];
        }
        // (given back only now: a slot is not handed on within the request that still uses it)
        for (int64_t j = j0; j < j1; ++j) {
            const int32_t slot = t->seg[(size_t)j].id;
            if (last_ref[(size_t)seg_at[(size_t)(j - j0)]] == r) free_slots.push_back(slot);
        }
    }
    t->n_slots = n_slots;
    return segments_suit(t) ? GORGO_OK : block_rows(t, keys);
}

int check_and_finish(gorgo_trace* t, const std::vector<IdRun>& runs, int32_t block_tokens) {
    if (block_tokens < 1) return fail(GORGO_ERR_INVALID_ARG, "block_tokens must be >= 1");
    const int64_t N = t->N;
    if (N >= 0x7FFFFFFF) return fail(GORGO_ERR_INVALID_ARG, "too many requests (limit 2^31-2)");
    if (t->blk_off[0] != 0) return fail(GORGO_ERR_INVALID_ARG, "blk_off[0] must be 0");
    for (int64_t r = 0; r < N; ++r) {
        if (r > 0 && t->ts[r] < t->ts[r - 1])
            return fail(GORGO_ERR_UNSORTED, "timestamps decrease at request " + std::to_string(r));
        if (t->ts[r] < 0) return fail(GORGO_ERR_INVALID_ARG, "negative timestamp at request " + std::to_string(r));
        if (t->ts[r] > (int64_t)1 << 53) return fail(GORGO_ERR_INVALID_ARG, "timestamp above 2^53 ms");
        if (t->in_len[r] < 0 || t->out_len[r] < 0)
            return fail(GORGO_ERR_INVALID_ARG, "negative token count at request " + std::to_string(r));
        const int64_t n = t->blk_off[r + 1] - t->blk_off[r];
        if (n < 0) return fail(GORGO_ERR_INVALID_ARG, "blk_off decreases at request " + std::to_string(r));
        if (n > 65535) return fail(GORGO_ERR_INVALID_ARG, "more than 65535 blocks in request " + std::to_string(r));
    }
    // the load signal (sum of input tokens in flight) is carried in fp64 and must stay an exact integer
    int64_t total_tokens = 0;
    for (int64_t r = 0; r < N; ++r) {
        total_tokens += t->in_len[r];
        if (total_tokens > ((int64_t)1 << 53)) return fail(GORGO_ERR_INVALID_ARG, "input tokens sum above 2^53");
    }
    t->block_tokens = block_tokens;
    // session-affinity policy (Sec. 4 "Baseline policies"): hash of the request's first block, here the high word
    // of the output that a SplitMix64 generator (Steele, Lea, Flood, OOPSLA'14) in state `id` gives next
    t->first_hash.assign((size_t)N, 0u);
    Ids ids(runs);
    for (int64_t r = 0; r < N; ++r)
        if (t->blk_off[r + 1] > t->blk_off[r]) {
            uint64_t z = (uint64_t)*ids.of(t->blk_off[r]) + 0x9E3779B97F4A7C15ull;
            z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
            z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
            t->first_hash[(size_t)r] = (uint32_t)((z ^ (z >> 31)) >> 32);
        }
    return preprocess(t, runs);
}

// ---- minimal JSON scanner (enough for flat objects with numbers, strings and arrays of numbers)
struct Cur {
    const char* p;
    const char* e;
    void ws() { while (p < e && (*p == ' ' || *p == '\t' || *p == '\r')) ++p; }
};

bool parse_int(Cur& c, int64_t* out) {
    c.ws();
    const char* s = c.p;
    bool neg = false;
    if (c.p < c.e && (*c.p == '-' || *c.p == '+')) { neg = *c.p == '-'; ++c.p; }
    if (c.p >= c.e || *c.p < '0' || *c.p > '9') { c.p = s; return false; }
    uint64_t v = 0;
    while (c.p < c.e && *c.p >= '0' && *c.p <= '9') {
        if (v > (std::numeric_limits<uint64_t>::max() - 9) / 10) return false;
        v = v * 10 + (uint64_t)(*c.p - '0');
        ++c.p;
    }
    // accept an integral float such as 12.0 or 1e3 only if it has no fractional/exponent part
    if (c.p < c.e && (*c.p == '.' || *c.p == 'e' || *c.p == 'E')) {
        char* endp = nullptr;
        std::string tmp(s, (size_t)std::min<ptrdiff_t>(c.e - s, 64));
        double d = std::strtod(tmp.c_str(), &endp);
        if (endp == tmp.c_str() || d != (double)(int64_t)d) return false;
        c.p = s + (endp - tmp.c_str());
        *out = (int64_t)d;
        return true;
    }
    if (!neg && v > (uint64_t)std::numeric_limits<int64_t>::max()) return false;
    *out = neg ? -(int64_t)v : (int64_t)v;
    return true;
}

bool skip_string(Cur& c) {
    if (c.p >= c.e || *c.p != '"') return false;
    ++c.p;
    while (c.p < c.e && *c.p != '"') {
        if (*c.p == '\\') ++c.p;
        ++c.p;
    }
    if (c.p >= c.e) return false;
    ++c.p;
    return true;
}

bool skip_value(Cur& c, int depth = 0) {
    c.ws();
    if (c.p >= c.e || depth > 32) return false;
    if (*c.p == '"') return skip_string(c);
    if (*c.p == '{' || *c.p == '[') {
        const char close = *c.p == '{' ? '}' : ']';
        const bool obj = *c.p == '{';
        ++c.p;
        c.ws();
        if (c.p < c.e && *c.p == close) { ++c.p; return true; }
        for (;;) {
            if (obj) {
                c.ws();
                if (!skip_string(c)) return false;
                c.ws();
                if (c.p >= c.e || *c.p != ':') return false;
                ++c.p;
            }
            if (!skip_value(c, depth + 1)) return false;
            c.ws();
            if (c.p < c.e && *c.p == ',') { ++c.p; continue; }
            if (c.p < c.e && *c.p == close) { ++c.p; return true; }
            return false;
        }
    }
    // number / true / false / null
    const char* s = c.p;
    while (c.p < c.e && *c.p != ',' && *c.p != '}' && *c.p != ']' && *c.p != ' ' && *c.p != '\t') ++c.p;
    return c.p > s;
}

// Parses one record.  Returns false on malformed input.
bool parse_line(const char* b, const char* e, int64_t* ts, int64_t* il, int64_t* ol, std::vector<int64_t>* ids,
                unsigned* have) {
    Cur c{b, e};
    c.ws();
    if (c.p >= c.e || *c.p != '{') return false;
    ++c.p;
    *have = 0;
    c.ws();
    if (c.p < c.e && *c.p == '}') return true;
    for (;;) {
        c.ws();
        const char* ks = c.p;
        if (!skip_string(c)) return false;
        std::string key(ks + 1, c.p - 1);
        c.ws();
        if (c.p >= c.e || *c.p != ':') return false;
        ++c.p;
        if (key == "timestamp") { if (!parse_int(c, ts)) return false; *have |= 1; }
        else if (key == "input_length") { if (!parse_int(c, il)) return false; *have |= 2; }
        else if (key == "output_length") { if (!parse_int(c, ol)) return false; *have |= 4; }
        else if (key == "hash_ids") {
            c.ws();
            if (c.p >= c.e || *c.p != '[') return false;
            ++c.p;
            c.ws();
            if (c.p < c.e && *c.p == ']') { ++c.p; }
            else {
                for (;;) {
                    int64_t v;
                    if (!parse_int(c, &v)) return false;
                    ids->push_back(v);
                    c.ws();
                    if (c.p < c.e && *c.p == ',') { ++c.p; continue; }
                    if (c.p < c.e && *c.p == ']') { ++c.p; break; }
                    return false;
                }
            }
            *have |= 8;
        } else if (!skip_value(c)) return false;
        c.ws();
        if (c.p < c.e && *c.p == ',') { ++c.p; continue; }
        if (c.p < c.e && *c.p == '}') { ++c.p; break; }
        return false;
    }
    c.ws();
    return c.p == c.e;
}

// Records of a piece of a file; `off` begins with the 0 of the first one.  The block ids of pieces behind the first stay where
// they were parsed (`more`), each from where its first request's begin.
struct Records {
    struct More {
        int64_t from;
        std::vector<int64_t> ids;
    };
    std::vector<More> more;
    std::vector<int64_t> ts, off{0}, ids;
    std::vector<int32_t> in_len, out_len;
    int64_t lines = 0;           // read so far
    int rc = GORGO_OK;           // what ended it: about its last line, where that is to be told
    const char* what = nullptr;

    // one line; false: stop
    bool add(const char* b, const char* e) {
        ++lines;
        const char* a = b;
        while (a < e && (*a == ' ' || *a == '\t' || *a == '\r')) ++a;
        if (a == e) return true;                  // blank
        int64_t t0 = 0, i0 = 0, o0 = 0;
        unsigned have = 0;
        rc = GORGO_ERR_PARSE;
        if (!parse_line(b, e, &t0, &i0, &o0, &ids, &have)) return false;
        what = ": needs timestamp, input_length, output_length and hash_ids";
        if (have != 15u) return false;
        what = ": token count out of range";
        if (i0 < 0 || i0 > 0x7FFFFFFF || o0 < 0 || o0 > 0x7FFFFFFF) return false;
        rc = GORGO_OK;
        what = nullptr;
        ts.push_back(t0);
        in_len.push_back((int32_t)i0);
        out_len.push_back((int32_t)o0);
        off.push_back((int64_t)ids.size());
        return true;
    }
    // whole lines, the last with or without its end
    void parse(const char* b, const char* e) {
        try {
            while (b < e) {
                const char* nl = static_cast<const char*>(std::memchr(b, '\n', (size_t)(e - b)));
                if (!add(b, nl ? nl : e)) return;
                b = nl ? nl + 1 : e;
            }
        } catch (const std::bad_alloc&) {
            rc = GORGO_ERR_OOM;
        }
    }
    // the same where there are NULs, which end what is read of a line, or of LINE_PART bytes of it, but not the line
    static constexpr size_t LINE_PART = (1 << 16) - 1;
    void parse_with_nuls(const char* b, const char* e) {
        try {
            std::string line;
            for (bool more = true; more;) {
                line.clear();
                for (;;) {
                    if (b >= e) { more = false; break; }
                    const size_t most = std::min((size_t)(e - b), LINE_PART);
                    const char* nl = static_cast<const char*>(std::memchr(b, '\n', most));
                    const size_t part = nl ? (size_t)(nl - b) + 1 : most, n = strnlen(b, part);
                    const bool whole = n > 0 && b[n - 1] == '\n';
                    line.append(b, whole ? n - 1 : n);
                    b += part;
                    if (whole) break;
                }
                if (!add(line.data(), line.data() + line.size())) return;
            }
        } catch (const std::bad_alloc&) {
            rc = GORGO_ERR_OOM;
        }
    }
    void append(Records& x) {
        if (lines == 0) {
            *this = std::move(x);
            return;
        }
        const int64_t at = off.back();
        ts.insert(ts.end(), x.ts.begin(), x.ts.end());
        in_len.insert(in_len.end(), x.in_len.begin(), x.in_len.end());
        out_len.insert(out_len.end(), x.out_len.begin(), x.out_len.end());
        for (size_t i = 1; i < x.off.size(); ++i) off.push_back(at + x.off[i]);
        if (x.off.back() > 0) more.push_back(More{at, std::move(x.ids)});
        lines += x.lines;
        rc = x.rc;
        what = x.what;
    }
};

// A file of records, in blocks of whole lines, a block in as many pieces as there are threads for it.  (A file of 5,000 requests
// and 319,000 block ids, 2.6 MB: 4.7 ms to load with one thread and a copy of every line; 3.3 with the pieces' ids put together
// in one array, 2.4 without, and with what stands at IdMap and below about the numbering, 1.3 of it, and the segments.)
#ifndef GORGO_READ_BYTES       // (tests read small files in blocks and pieces of a few lines)
#define GORGO_READ_BYTES ((size_t)32 << 20)
#define GORGO_PIECE_BYTES ((size_t)128 << 10)
#endif
constexpr size_t READ_BYTES = GORGO_READ_BYTES, PIECE_BYTES = GORGO_PIECE_BYTES;
constexpr unsigned READ_THREADS = 8;

int read_records(FILE* f, const char* path, Records* all) {
    try {
        std::vector<Records> piece;
        size_t room = READ_BYTES, have = 0;      // bytes in hand, of the last block's last line to begin with
        struct stat st;
        if (fstat(fileno(f), &st) == 0 && S_ISREG(st.st_mode) && (size_t)st.st_size < room) room = (size_t)st.st_size + 1;
        std::unique_ptr<char[]> text(new char[room]);
        bool nuls = false;
        for (bool end = false; !end;) {
            have += std::fread(text.get() + have, 1, room - have, f);
            const bool failed = std::ferror(f) != 0;
            end = failed || have < room;
            const char *b = text.get(), *e = b + have;
            nuls = nuls || std::memchr(b, 0, have);
            if (!end || failed) {
                const char* nl = static_cast<const char*>(memrchr(b, '\n', have));
                e = nl && !nuls ? nl + 1 : b;     // (with NULs the rest of the file is read first)
                if (failed && nuls) e = nl ? nl + 1 : b;
            }
            if (nuls) {
                Records rest;
                if (b < e) rest.parse_with_nuls(b, e);      // (nothing is not a line)
                all->append(rest);
            } else {
                const size_t bytes = (size_t)(e - b);
                const size_t most = std::min(std::max(1u, std::thread::hardware_concurrency()), READ_THREADS);
                const size_t n = std::min(most, bytes / PIECE_BYTES + 1);
                piece.assign(n, Records());
                std::vector<std::thread> threads;
                threads.reserve(n);
                const char* from = b;
                for (size_t i = 0; i < n; ++i) {
                    const char* to = e;
                    if (i + 1 < n) {
                        to = std::max(from, b + bytes / n * (i + 1));
                        const char* nl = static_cast<const char*>(std::memchr(to, '\n', (size_t)(e - to)));
                        to = nl ? nl + 1 : e;
                    }
                    auto parse = [&piece, i, from, to] { piece[i].parse(from, to); };
                    bool started = false;
                    if (i + 1 < n) {
                        try {
                            threads.emplace_back(parse);
                            started = true;
                        } catch (const std::exception&) {       // (no thread to be had: here, then)
                        }
                    }
                    if (!started) parse();
                    from = to;
                }
                for (std::thread& t : threads) t.join();
                for (size_t i = 0; i < n && all->rc == GORGO_OK; ++i) all->append(piece[i]);
            }
            if (all->rc == GORGO_ERR_OOM) return fail(GORGO_ERR_OOM, "out of host memory");
            if (all->rc != GORGO_OK)
                return fail(all->rc, (all->what ? "line " : "malformed record on line ") + std::to_string(all->lines) +
                                         (all->what ? all->what : ""));
            if (failed) return fail(GORGO_ERR_IO, std::string("read error on ") + path);
            have = (size_t)(text.get() + have - e);
            std::memmove(text.get(), e, have);
            if (!end && have == room) {           // (a line longer than a block)
                std::unique_ptr<char[]> larger(new char[2 * room]);
                std::memcpy(larger.get(), text.get(), have);
                text.swap(larger);
                room *= 2;
            }
        }
    } catch (const std::bad_alloc&) {
        return fail(GORGO_ERR_OOM, "out of host memory");
    }
    return GORGO_OK;
}

}  // namespace
}  // namespace gorgo

using namespace gorgo;

extern "C" {

const char* gorgo_last_error(void) { return g_err.c_str(); }

int gorgo_load_trace_arrays(int64_t N, const int64_t* ts_ms, const int32_t* in_len, const int32_t* out_len,
                            const int64_t* blk_off, const int64_t* hash_ids, int32_t block_tokens,
                            gorgo_trace** out) {
    clear_error();
    if (!out) return fail(GORGO_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (N < 0) return fail(GORGO_ERR_INVALID_ARG, "N is negative");
    if (!blk_off) return fail(GORGO_ERR_INVALID_ARG, "blk_off is NULL");
    if (N > 0 && (!ts_ms || !in_len || !out_len)) return fail(GORGO_ERR_INVALID_ARG, "a request array is NULL");
    if (N >= 0x7FFFFFFF) return fail(GORGO_ERR_INVALID_ARG, "too many requests (limit 2^31-2)");
    if (N > 0 && blk_off[N] > 0 && !hash_ids) return fail(GORGO_ERR_INVALID_ARG, "hash_ids is NULL");
    gorgo_trace* t = new (std::nothrow) gorgo_trace();
    if (!t) return fail(GORGO_ERR_OOM, "out of host memory");
    try {
        t->N = N;
        t->ts.assign(ts_ms, ts_ms + N);
        t->in_len.assign(in_len, in_len + N);
        t->out_len.assign(out_len, out_len + N);
        t->blk_off.assign(blk_off, blk_off + N + 1);
        int rc = check_and_finish(t, {IdRun{0, hash_ids}}, block_tokens);
        if (rc != GORGO_OK) { delete t; return rc; }
    } catch (const std::bad_alloc&) {
        delete t;
        return fail(GORGO_ERR_OOM, "out of host memory");
    }
    *out = t;
    return GORGO_OK;
}

int gorgo_load_trace(const char* jsonl_path, int32_t block_tokens, gorgo_trace** out) {
    clear_error();
    if (!out) return fail(GORGO_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (!jsonl_path) return fail(GORGO_ERR_INVALID_ARG, "path is NULL");
    FILE* f = std::fopen(jsonl_path, "rb");
    if (!f) return fail(GORGO_ERR_IO, std::string("cannot open ") + jsonl_path + ": " + std::strerror(errno));
    Records all;
    int rc = read_records(f, jsonl_path, &all);
    std::fclose(f);
    if (rc != GORGO_OK) return rc;
    gorgo_trace* t = new (std::nothrow) gorgo_trace();
    if (!t) return fail(GORGO_ERR_OOM, "out of host memory");
    try {
        std::vector<IdRun> runs{IdRun{0, all.ids.data()}};
        for (const Records::More& x : all.more) runs.push_back(IdRun{x.from, x.ids.data()});
        t->N = (int64_t)all.ts.size();
        t->ts = std::move(all.ts);
        t->in_len = std::move(all.in_len);
        t->out_len = std::move(all.out_len);
        t->blk_off = std::move(all.off);
        rc = check_and_finish(t, runs, block_tokens);
    } catch (const std::bad_alloc&) {
        rc = fail(GORGO_ERR_OOM, "out of host memory");
    }
    if (rc != GORGO_OK) { delete t; return rc; }
    *out = t;
    return GORGO_OK;
}

int gorgo_trace_info(const gorgo_trace* t, int64_t* N, int64_t* total_blocks, int32_t* max_blocks,
                     int64_t* unique_ids, int32_t* chain_consistent) {
    clear_error();
    if (!t) return fail(GORGO_ERR_INVALID_ARG, "trace is NULL");
    if (N) *N = t->N;
    if (total_blocks) *total_blocks = t->total_blocks;
    if (max_blocks) *max_blocks = t->max_blocks;
    if (unique_ids) *unique_ids = t->unique_ids;
    if (chain_consistent) *chain_consistent = t->chain_consistent ? 1 : 0;
    return GORGO_OK;
}

void gorgo_free_trace(gorgo_trace* t) {
    if (!t) return;
    release_device_trace(t);
    delete t;
}

}  // extern "C"

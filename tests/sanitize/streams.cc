// CPU-only check program, built by tests/test_stream_bounds.py with -fsanitize=address,undefined: the stream readers and the
// decoders of huff_decode.cuh and tree_walk.cuh, compiled for the CPU lane by lane, over records of the oracle's encoder that
// end kStreamSlack bytes in front of the end of their allocation.  Every read behind that (or in front of the record) is a
// sanitizer report, and every code has to come out.  The arena's layout is checked to leave as much behind the last record
// that fits, and a staging area to hold the records that it may meet.  Exit status 0 = all checks passed.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "../../paper_2509_00579_amd/csrc/host_logic.h"
#include "../../paper_2509_00579_amd/csrc/huff_decode.cuh"
#include "../../paper_2509_00579_amd/csrc/tree_walk.cuh"

extern "C" {
size_t orc_encode_block(int which, int k_mode, const uint8_t *codes, const uint16_t *minmax, const uint8_t *len,
                        const uint32_t *code, uint8_t *rec, size_t cap);
}

#define CHECK(cond)                                                                 \
    do {                                                                            \
        if (!(cond)) {                                                              \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            std::exit(1);                                                           \
        }                                                                           \
    } while (0)

using namespace kvc;
using namespace kvc::host;

// A record, and behind it kStreamSlack bytes and nothing else
struct Record {
    std::vector<uint8_t> bytes;
    uint8_t *mem;
    int which, hdr;
    explicit Record(const std::vector<uint8_t> &rec, int w, int h) : bytes(rec), mem(nullptr), which(w), hdr(h) {
        const size_t n = rec.size() + kStreamSlack;
        CHECK(rec.size() % 16 == 0 && posix_memalign(reinterpret_cast<void **>(&mem), 16, n) == 0);
        std::memcpy(mem, rec.data(), rec.size());
        std::memset(mem + rec.size(), 0xA5, kStreamSlack);
    }
    ~Record() { std::free(mem); }
    const Unit *units() const { return payload_units(reinterpret_cast<const uint32_t *>(mem + hdr)); }
    uint32_t bits(int slice) const {
        uint16_t b;
        std::memcpy(&b, mem + hdr - 2 * kSlices + 2 * slice, 2);
        return b;
    }
    uint32_t start(int slice) const {
        uint32_t at = 0;
        for (int s = 0; s < slice; s++) at += bits(s);
        return at;
    }
};
// code `pos` of slice s in a token-major block
static int code_at(int which, int s, int pos) { return which == 0 ? s * kSliceLen + pos : pos * kD + s; }

struct Book {
    uint8_t len[256];
    uint32_t code[256];
    std::vector<uint32_t> enc, pair;
    std::vector<uint16_t> lut;
    std::vector<int16_t> tree;
    int bits;
    Book(const uint32_t *hist, int n_sym, int limit) : enc(512), pair(kPairTableEntries), lut(kLutSize), tree(512) {
        build_codebook_host(hist, n_sym, limit, len, code);
        bits = build_tables(len, code, enc.data(), lut.data(), tree.data());
        if (bits <= 6) build_pair_table(lut.data(), bits, pair.data());
    }
};

template <int LB>
static void decode(const Record &r, const Book &book, const std::vector<uint8_t> &codes) {
    using M = DecodeMode<LB>;
    const char *lut = M::kPair ? reinterpret_cast<const char *>(book.pair.data()) : reinterpret_cast<const char *>(book.lut.data());
    const uint32_t mask = M::kPair ? ((1u << kPairIndexBits) - 1u) << 2 : ((1u << book.bits) - 1u) << 1;
    for (int lane = 0; lane < 64; lane++) {
        for (int apart = 0; apart < 2; apart++) {  // neighbouring slices, and slices lane and lane + 64
            const int sa = apart ? lane : 2 * lane, sb = apart ? lane + 64 : 2 * lane + 1;
            Quad<M::J> qd;
            if (apart) qd.open2(r.units(), r.start(sa), r.bits(sa), r.start(sb), r.bits(sb));
            else qd.open(r.units(), r.start(sa), r.bits(sa), r.bits(sb));
            SliceWords pw;
            decode_block<LB>(qd, r.units(), lut, mask, pw);
            for (int i = 0; i < kSliceLen; i++) {
                CHECK(((pw.a[i / 4] >> (8 * (i % 4))) & 0xffu) == codes[code_at(r.which, sa, i)]);
                CHECK(((pw.b[i / 4] >> (8 * (i % 4))) & 0xffu) == codes[code_at(r.which, sb, i)]);
            }
        }
    }
}

// the bit-serial walk, as long as the slowest lane of a wave may keep the others going
static void walk(const Record &r, const Book &book, const std::vector<uint8_t> &codes) {
    for (int lane = 0; lane < 64; lane++) {
        const int sa = 2 * lane;
        int emitted = 0;
        walk_chains(r.units(), book.tree.data(), r.start(sa), r.bits(sa), r.bits(sa + 1),
                    [&](int c, int sym, int idx) {
                        if (sym < 0) return;
                        CHECK(sym == codes[code_at(r.which, sa + (c >> 1), (c & 1) ? kSliceLen - 1 - idx : idx)]);
                        emitted++;
                    },
                    [](bool) { return true; });
        CHECK(emitted == 2 * kSliceLen);
    }
}

static void records(std::mt19937_64 &rng) {
    int cases = 0;
    for (int round = 0; round < 120; round++) {
        const int which = round & 1, k_mode = which == 0 ? (round >> 1) & 1 : 0;
        const int n_sym = round % 3 == 0 ? 2 + (int)(rng() % 7) : 2 + (int)(rng() % 255);
        int min_limit = 1;
        while ((1 << min_limit) < n_sym) min_limit++;
        const int limit = min_limit + (int)(rng() % (kLutBits - min_limit + 1));
        // a steep histogram: code words from one bit up to the limit
        uint32_t hist[256] = {0};
        for (int s = 0; s < n_sym; s++) hist[s] = 1u + (0x40000000u >> (s < 30 ? s : 30));
        const Book book(hist, n_sym, limit);
        int longest = 0;
        for (int s = 0; s < n_sym; s++) longest = book.len[s] > book.len[longest] ? s : longest;
        // slices of the shortest code words, of the longest, and of both kinds mixed, the kinds in another order every round
        std::vector<uint8_t> codes(kTile);
        for (int s = 0; s < kSlices; s++) {
            const int kind = round < 12 ? round / 4 : (int)(rng() % 4);
            for (int i = 0; i < kSliceLen; i++)
                codes[code_at(which, s, i)] = (uint8_t)(kind == 0 ? 0 : kind == 1 ? longest : kind == 2 ? (int)(rng() % n_sym) : (rng() % 16 ? 0 : longest));
        }
        const int hdr = which ? kHdrBytesV : (k_mode ? 16 : kMinMaxBytesK) + 2 * kSlices;
        std::vector<uint16_t> minmax(2 * 128, 0);
        std::vector<uint8_t> rec((size_t)hdr + kMaxPayloadBytes + 16);
        const size_t n = orc_encode_block(which, k_mode, codes.data(), minmax.data(), book.len, book.code, rec.data(), rec.size());
        CHECK(n > 0 && n <= rec.size());
        rec.resize((n + 15) / 16 * 16);
        const Record r(rec, which, hdr);
        if (book.bits <= 6) decode<6>(r, book, codes);
        if (book.bits <= 7) decode<7>(r, book, codes);
        if (book.bits <= 8) decode<8>(r, book, codes);
        if (book.bits <= 10) decode<10>(r, book, codes);
        decode<12>(r, book, codes);
        walk(r, book, codes);
        cases++;
    }
    std::printf("records: %d\n", cases);
}

static void arena() {
    int cases = 0;
    for (int B : {1, 3}) for (int H : {1, 2, 8}) for (int seq : {64, 100, 128, 1000, 4096}) for (int k_mode : {0, 1})
        for (int limit : {0, 6, 7, 9, 12}) {
            const kvcomp_config c = {B, H, H, 128, 64, seq, 1e-2f, 1e-2f, k_mode, limit, 0};
            CHECK(valid_cfg(&c));
            const Layout L = make_layout(c);
            const size_t records_end = L.payload + L.payload_cap16 * 16;  // of the last record that a placement admits
            CHECK(records_end + kStreamSlack <= L.total);
            const size_t worst_k = align_up((size_t)k_header_bytes(c) + (size_t)kTile * code_len_limit(c) / 8, 16);
            const size_t worst_v = align_up(kHdrBytesV + (size_t)kTile * code_len_limit(c) / 8, 16);
            CHECK(L.payload_cap16 * 16 >= (size_t)B * H * (seq / 64) * (worst_k + worst_v));
            cases++;
        }
    std::printf("arenas: %d\n", cases);
}

static void staging() {
    for (uint32_t size16 = 0; size16 <= (uint32_t)kMaxRecordBytes / 16; size16++) {
        const int known = stage_bytes_for(size16, false), flushed = stage_bytes_for(size16, true);
        CHECK(known % 16 == 0 && flushed % 16 == 0);
        CHECK((known - kStreamSlack) / 16 >= (int)size16);           // the largest record fits
        CHECK((flushed - kStreamSlack) / 16 >= (int)size16 + 8);     // and behind a flush one that is 128 bytes longer
    }
}

int main() {
    std::mt19937_64 rng(20250908);
    records(rng);
    arena();
    staging();
    std::printf("streams driver: ok\n");
    return 0;
}

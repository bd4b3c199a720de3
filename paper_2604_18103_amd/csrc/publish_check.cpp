// Host-side check of the exchanges between the workgroups of the one-launch score + decision + compaction kernels (test
// infrastructure, CPU only; part of the same small library as staging_check.cpp). Steps the kernels' protocols with the words and
// functions that they use (publish.h).
#include <vector>

#include "publish.h"

using namespace dash;

extern "C" {

// Steps the exchange of the one-launch NONE / THRESHOLD kernel over `chunks` chunks of 64 rows and `splits` column splits; chunk c keeps
// c % 65 rows. late >= 0: that chunk's publisher comes only after everybody that waits for its words has given up. backwards: the
// others run from the last chunk to the first. Returns the survivor count; gathered[c]: how many of chunk c's workgroups gathered rows.
int dash_check_publish(int chunks, int splits, int late, int backwards, int* gathered) {
    std::vector<unsigned long long> words((size_t)chunks * 2, 0);
    auto mask_of = [](int c) { return c % 65 == 64 ? ~0ull : (1ull << (c % 65)) - 1; };
    auto publish = [&](int c) {
        words[2 * c] = pub_word0(mask_of(c), c % 65);
        words[2 * c + 1] = pub_word1(mask_of(c));
    };
    for (int c = 0; c < chunks; ++c) {  // publishers wait for nothing before they publish
        gathered[c] = 0;
        if (c != late) publish(c);
    }
    int n_out = 0, wrong = 0;
    auto rest_of = [&](int c, int y) {  // what a workgroup does once its own mask is there, or not
        bool bad = y > 0 && !(pub_ready(words[2 * c]) && pub_ready(words[2 * c + 1]));
        int base = 0;
        for (int e = 0; e < c; ++e) {
            bad = bad || !pub_ready(words[2 * e]);
            base += pub_count(words[2 * e]);
        }
        if (bad) {
            n_out = -1;
            return;
        }
        if (y > 0 && pub_mask(words[2 * c], words[2 * c + 1]) != mask_of(c)) wrong = 1;
        ++gathered[c];
        if (c == chunks - 1 && y == 0 && n_out == 0) n_out = base + c % 65;  // exchanges the 0
    };
    for (int i = 0; i < chunks; ++i) {
        const int c = backwards ? chunks - 1 - i : i;
        for (int y = 0; y < splits; ++y)
            if (c != late || y > 0) rest_of(c, y);
    }
    if (late >= 0) {
        publish(late);
        rest_of(late, 0);
    }
    return wrong ? -100 : n_out;
}

// Steps the keys' way into every thread of a one-launch TopK workgroup over n rows (take_keys); the words of rows [late0, late1) are still 0
// the first late_asks times a thread asks for them (below 0: every time). *own: rows whose key was made from the pairs. Returns how
// many rows ended with another key than their own.
int dash_check_topk_keys(int n, int late0, int late1, int late_asks, int* own) {
    constexpr int kStride = 1024, B = 4;
    auto key_of = [](int r) { return 0x80000000u + 2654435761u * (uint32_t)r % 0x7FFFFFFFu; };
    int wrong = 0;
    *own = 0;
    for (int tid = 0; tid < kStride; ++tid) {
        std::vector<int> asked((size_t)n, 0);
        uint32_t key[B];
        take_keys<B>(
            key, tid, kStride, n,
            [&](int r) { return r >= late0 && r < late1 && (late_asks < 0 || asked[(size_t)r]++ < late_asks) ? 0u : key_of(r); },
            [&](int r) { ++*own; return key_of(r); }, [] {});
        for (int u = 0; u < B; ++u) wrong += key[u] != (u * kStride + tid < n ? key_of(u * kStride + tid) : 0u);
    }
    return wrong;
}
int dash_key_asks() { return kKeyAsks; }

}  // extern "C"

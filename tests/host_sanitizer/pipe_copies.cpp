// The copies of a wavefront of linear_pipe.hip, chunk by chunk, against the waits that are to have brought them in.  A wait for all but n
// leaves the n youngest copies of the queue under way, nothing more is assumed.  Two queues: one in which copies of no lanes take no
// place, one in which they do.  Exit status 1 if a chunk reads something that has not landed.
#include <cstdio>
#include <string>
#include <vector>

#include "../../paper_2505_14638_amd/csrc/pipe_copies.hpp"

namespace {

struct Copy {
    char kind;      // p: page of activations, s: scales, r: nibbles, e: record
    int chunk;
    bool real;
};

int failures = 0;

// pages, scales, records: copies of each per chunk (one of nibbles); n: chunks of the K range
void run(int pages, int scales, int records, int n, bool empty_ones_count) {
    std::vector<Copy> under_way;
    auto issue = [&](char kind, int count, int chunk) {
        const Copy c{kind, chunk, chunk < n};
        if (c.real || empty_ones_count) under_way.insert(under_way.end(), count, c);
    };
    auto wait = [&](int left) {
        const size_t n_left = w4a8::copies_that_may_be_left(pages + scales, 1 + records, left);
        if (under_way.size() > n_left) under_way.erase(under_way.begin(), under_way.end() - n_left);
    };
    auto landed = [&](const char* kinds, int chunk, int at) {
        if (chunk >= n) return;
        for (const Copy& c : under_way)
            if (c.real && c.chunk == chunk && std::string(kinds).find(c.kind) != std::string::npos) {
                std::printf("%d chunks, %d pages: chunk %d reads %c of chunk %d\n", n, pages, at, c.kind, chunk);
                ++failures;
                return;
            }
    };
    // a tile's start: chunks 0 and 1, the nibbles and the record of chunk 2 (those of 0 and 1 come through registers); then the rest
    for (int c = 0; c < 2; ++c) {
        issue('p', pages, c);
        issue('s', scales, c);
    }
    issue('r', 1, 2);
    issue('e', records, 2);
    issue('p', pages, 2);
    issue('s', scales, 2);
    issue('r', 1, 3);
    issue('e', records, 3);
    wait(n + 1);
    landed("ps", 0, -1);
    for (int c = 0; c < n; ++c) {
        landed("ps", c + 1, c);
        landed("re", c + 2, c);
        issue('p', pages, c + 3);
        issue('r', 1, c + 4);
        issue('s', scales, c + 3);
        issue('e', records, c + 4);
        wait(n - c);
    }
}

}  // namespace

int main() {
    for (int pages : {2, 4})
        for (int scales : {0, 1})
            for (int records : {0, 1})
                for (int n = 1; n <= 12; ++n)
                    for (bool count : {false, true}) run(pages, scales, records, n, count);
    if (failures == 0) std::puts("all copies have landed");
    return failures != 0;
}

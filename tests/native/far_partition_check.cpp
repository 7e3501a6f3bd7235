// CPU check of the in-place partition's schedule (far_partition.h): lists read from standard input, one
// per line (0 near, 1 far), are partitioned step by step as k_far.hip does.  Prints for every line
// "near count|list afterwards|most ids held of one kind|0 or what went wrong".
#include <algorithm>
#include <cstdio>
#include <iostream>
#include <string>
#include <vector>

#include "far_partition.h"

using namespace fdx;

int main() {
    std::string line;
    while (std::getline(std::cin, line)) {
        const uint32_t ns = (uint32_t)line.size();
        std::vector<uint32_t> list(ns);
        std::vector<int> unread(ns, 1);
        for (uint32_t i = 0; i < ns; i++) list[i] = i;
        const char *wrong = "0";
        std::vector<uint32_t> ids(2 * kFarHeld);          // [kind][held], as in LDS
        uint32_t most = 0;
        FarPartition p(ns);
        using Block = FarPartition::Block;
        auto read = [&](const Block &b) {                 // a block's ids are read when it is chosen
            for (uint32_t i = 0; i < b.len; i++)
                if (!unread[b.start + i]) wrong = "a slot is read twice or after it was written";
            return std::vector<uint32_t>(list.begin() + b.start, list.begin() + b.start + b.len);
        };
        auto write = [&](int c, uint32_t i, uint32_t id) {
            const uint32_t s = p.slot(c, i);
            if (s >= ns || unread[s]) { wrong = "an unread slot is overwritten"; return; }
            list[s] = id;
        };
        Block b0 = p.choose(0), b1 = p.choose(0);
        std::vector<uint32_t> id0 = read(b0), id1 = read(b1);
        while (b0.len) {
            for (uint32_t v : id0) {
                const int c = line[v] == '1';
                if (p.held[c] >= kFarHeld) { wrong = "more ids than the buffer holds"; break; }
                ids[c * kFarHeld + p.held[c]++] = v;
            }
            for (uint32_t i = 0; i < b0.len; i++) unread[b0.start + i] = 0;
            most = std::max(most, std::max(p.held[0], p.held[1]));
            const Block b2 = p.choose(p.sorted(b0));
            b0 = b1;
            b1 = b2;
            id0 = id1;
            id1 = read(b1);
            for (int c = 0; c < 2; c++) {
                const uint32_t n = p.ready(c);
                for (uint32_t i = 0; i < n; i++) write(c, i, ids[c * kFarHeld + p.held[c] + i]);
                p.written(c, n);
            }
        }
        for (int c = 0; c < 2; c++)
            for (uint32_t i = 0; i < p.held[c]; i++) write(c, i, ids[c * kFarHeld + i]);
        std::printf("%u|", p.put[0] + p.held[0]);
        for (uint32_t v : list) std::printf("%u ", v);
        std::printf("|%u|%s\n", most, wrong);
    }
    return 0;
}

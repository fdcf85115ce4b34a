// Runs the deciding half of greedy suppression (resolve_rows, nms.hpp) on the CPU with the
// emulator of emu_main.cpp: one workgroup of 16 waves that wait for each other's decisions in
// LDS.  Input file: n, LG, then for every box the indices of the boxes of higher rank that it
// overlaps (count, indices).  The overlaps are laid out as overlap_rows leaves them, each list
// in a shuffled order.  Output file: n bytes, 1 for a kept box.  Waves that wait for each other
// in a circle would never end: the caller's time limit is the test of that.
#define EMU_CORE_ONLY
#include "emu_main.cpp"

#include <random>

#include "nms_resolve.inc"

using namespace rex;

template <int M, int LG> static void run(uint64_t *ws, int n, std::vector<uint64_t> &kept) {
    static ResolveSmem<M> sm;
    emu_register(&sm, sizeof sm);
    launch(1, kNmsResolveThreads, 0, [&] { resolve_rows<M, LG>(ws, n, sm); });
    kept.assign(sm.kept, sm.kept + (n + 63) / 64);
}

template <int LG> static void decide(uint64_t *ws, int n, std::vector<uint64_t> &kept) {
    if (n <= 1024) run<1, LG>(ws, n, kept);
    else run<3, LG>(ws, n, kept);
}

int main(int, char **argv) {
    FILE *f = std::fopen(argv[1], "rb");
    int32_t head[2];
    if (!f || std::fread(head, 4, 2, f) != 2) return 2;
    const int n = head[0], lg = head[1], nb = (n + 63) / 64;
    std::vector<uint64_t> ws(nms_words(n), 0x5a5a5a5a5a5a5a5aull);
    const NmsLists l = nms_lists(ws.data(), n);
    std::vector<std::vector<std::pair<uint64_t, uint16_t>>> lists(nb << lg);
    for (int i = 0; i < n; ++i) {
        int32_t cnt;
        if (std::fread(&cnt, 4, 1, f) != 1) return 2;
        std::vector<int32_t> js(cnt);
        if (cnt && std::fread(js.data(), 4, cnt, f) != size_t(cnt)) return 2;
        std::vector<uint64_t> words(nb, 0);
        for (int j : js) words[j >> 6] |= uint64_t(1) << (j & 63);
        const int ib = i >> 6;
        l.own[i] = words[ib];
        for (int w = 0; w < ib; ++w)
            if (words[w]) lists[(ib << lg) + (w & ((1 << lg) - 1))].push_back({words[w], uint16_t((i & 63) | w << 6)});
    }
    std::mt19937 rng(n);
    for (int q = 0; q < (nb << lg) && nb > 1; ++q) {
        std::shuffle(lists[q].begin(), lists[q].end(), rng);
        l.len[q] = static_cast<int32_t>(lists[q].size());
        const int base = nms_list_base(n, q >> lg, q & ((1 << lg) - 1), lg);
        for (size_t e = 0; e < lists[q].size(); ++e) {
            l.word[base + e] = lists[q][e].first;
            l.tag[base + e] = lists[q][e].second;
        }
    }
    std::vector<uint64_t> kept;
    if (lg == 1) decide<1>(ws.data(), n, kept);
    else decide<3>(ws.data(), n, kept);
    std::vector<uint8_t> out(n);
    for (int i = 0; i < n; ++i) out[i] = (kept[i >> 6] >> (i & 63)) & 1;
    FILE *o = std::fopen(argv[2], "wb");
    std::fwrite(out.data(), 1, n, o);
    std::fclose(o);
    std::printf("done\n");
    return 0;
}

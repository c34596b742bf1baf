// Host run of the fused launch's kernel: one workgroup of EMU_BLOCK threads takes
// every graph of the batch in argv[1] (counts G, P, N; pair and vertex offsets;
// pairs) with a workspace that starts as 0xAB bytes, and writes all outputs to
// argv[2].  fused_body.inc is the kernel's source, extracted from tc_fused.hip by
// the test.
#include "tc_internal.h"

std::atomic<int> emu_or[2];
thread_local int emu_or_turn = 0;

#include "fused_body.inc"

template <typename T> static std::vector<T> read(FILE *f, int64_t n) {
    std::vector<T> v(n);
    if ((int64_t)fread(v.data(), sizeof(T), n, f) != n) exit(2);
    return v;
}
template <typename T> static void write(FILE *f, const std::vector<T> &v) {
    if (fwrite(v.data(), sizeof(T), v.size(), f) != v.size()) exit(3);
}

int main(int, char **argv) {
    FILE *in = fopen(argv[1], "rb"), *out = fopen(argv[2], "wb");
    const auto c = read<int64_t>(in, 3);
    const int64_t G = c[0], P = c[1], N = c[2];
    const auto po = read<int64_t>(in, G + 1), vo = read<int64_t>(in, G + 1);
    const auto src = read<int32_t>(in, P), dst = read<int32_t>(in, P);
    const int64_t bytes =
        FUSED_HEADER + pair_region(P) + FUSED_VTX_BYTES * N + FUSED_GRAPH_BYTES * G;
    std::vector<unsigned char> ws(bytes, 0xAB);
    memset(ws.data(), 0, 4);  // k_fused_init
    std::vector<int32_t> eu(P, -7), ev(P, -7), st(G, 99);
    std::vector<uint64_t> sup(P, 77), tri(N, 77), num(N, 77), tg(G, 77);
    std::vector<int64_t> ne(G, -7);
    std::vector<double> tc(N, -7);
    FusedArgs a;
    a.src = src.data();
    a.dst = dst.data();
    a.pair_off = po.data();
    a.vtx_off = vo.data();
    a.order = nullptr;
    a.G = (int32_t)G;
    a.P = P;
    a.N = N;
    a.eu = eu.data();
    a.ev = ev.data();
    a.sup = sup.data();
    a.num_edges = ne.data();
    a.tri = tri.data();
    a.num = num.data();
    a.tc = tc.data();
    a.triG = tg.data();
    a.status = st.data();
    a.ws = ws.data();
    emu_launch(1, EMU_BLOCK, [&] { k_fused_graphs<EMU_BLOCK>(a); });
    write(out, eu), write(out, ev), write(out, sup), write(out, ne), write(out, tri);
    write(out, tg), write(out, num), write(out, tc), write(out, st);
    fclose(out);
    return 0;
}

// Host driver of the block kernels' code generation (built by the CPU tests
// with g++ under AddressSanitizer and UndefinedBehaviorSanitizer, from
// construct.cpp, graph.cpp, codegen.cpp and abi.cpp).
//
// argv: "source KERNELS MOMENTUM" writes the generated source of the block
// adjoint (KERNELS 8192, several rows apart 65536; at complex energies 16384) or the block forward (32768)
// to stdout; "override" takes a handle's waves per block, then changes
// AMIGPU_JIT_BLOCK_WAVES and prints the count, the count asked for again and the
// one in the source.  stdin: "n_g n_eps n_freq n_int" and the alpha and eps
// entries row-major.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/amigpu.h"
#include "../../paper_2311_17189_amd/csrc/ami_internal.hpp"
#include "../../paper_2311_17189_amd/csrc/jit.hpp"

namespace ami {
AmiStatus code_from_source(const std::string &, std::vector<char> &, std::string &err) {
    err = "no run-time compiler in the host check";
    return AMI_E_UNSUPPORTED;
}
}  // namespace ami

extern "C" void amiFree(AmiTerms *t) { delete t; }

int main(int argc, char **argv) {
    int ng, ne, nf, ni;
    if (argc < 2 || std::scanf("%d %d %d %d", &ng, &ne, &nf, &ni) != 4) return 2;
    std::vector<int8_t> alpha(static_cast<size_t>(ng) * nf), eps(static_cast<size_t>(ng) * ne);
    for (auto *m : {&alpha, &eps})
        for (auto &x : *m) {
            int v;
            if (std::scanf("%d", &v) != 1) return 2;
            x = static_cast<int8_t>(v);
        }
    AmiTerms *t = nullptr;
    if (amiConstruct(ng, ne, nf, ni, alpha.data(), eps.data(), nullptr, 0, &t) != AMI_OK) return 3;
    if (std::strcmp(argv[1], "source") == 0 && argc == 4) {
        const int kernels = std::atoi(argv[2]);
        const bool hub = std::atoi(argv[3]) != 0;
        const int waves = kernels == 32768 ? ami::jit_block_forward_waves(t)
                                           : ami::jit_block_waves(t, hub, kernels == 16384, kernels == 65536);
        if (waves > 0) std::fputs(ami::jit_source(t, hub, kernels).c_str(), stdout);
    } else {
        const int first = ami::jit_block_waves(t, true, false);
        setenv("AMIGPU_JIT_BLOCK_WAVES", first == 4 ? "2" : "4", 1);
        const int again = ami::jit_block_waves(t, true, false);
        const std::string src = ami::jit_source(t, true, 8192);
        const size_t at = src.find("constexpr int NW = ");
        std::printf("%d %d %d\n", first, again, at == std::string::npos ? -1 : std::atoi(src.c_str() + at + 19));
    }
    amiFree(t);
    return 0;
}

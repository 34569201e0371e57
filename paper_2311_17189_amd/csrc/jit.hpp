// Run-time specialized evaluator: source generation (codegen.cpp) and its
// compilation, caching and loading (jit.cpp).
#pragma once

#include <string>
#include <vector>

#include "ami_internal.hpp"

namespace ami {

// Largest solution (flat terms) specialized; larger ones stay on the
// table-driven kernels, whose code size does not grow with the diagram.
constexpr int kJitMaxTerms = 1024;
// Largest solution evaluated by the two-pass specialized forward (group sums
// stored per sample by a first kernel, read back per frequency by a second):
// its register use does not grow with the number of groups.
constexpr int kJitTwoPassMaxTerms = 4096;
// AMI_VARIANT_AUTO uses the one-pass specialized adjoint up to this many
// terms: beyond it the straight-line reverse sweep outgrows the register file,
// and the adjoint runs in passes over a workspace (up to kJitTwoPassMaxTerms).
constexpr int kJitAutoAdjointTerms = 128;
// The same switch for the adjoint at complex energies, whose passes hold
// complex values per leaf and node (per 10^6-sample step: 264 terms one pass
// 0.91 ms, passes 1.75 ms; 380: 1.30 / 3.18 ms; 560: 2.21 / 1.91 ms).
constexpr int kJitAutoComplexAdjointTerms = 512;
// AUTO takes the block adjoint at complex energies above this many terms (2 10^5
// samples, one row: 264 terms one pass 205 us, block 110; 560: passes 302, block
// 137; four rows of 5 10^4: 91 and 55, 170 and 72), and with one frequency row
// from fewer on (136 terms 84 and 66 us, 76: 137 and 64, 52: 49.5 and 48.7, at 2 10^4
// samples 21.4 and 19.3).  With several rows each wave forms its denominators again for
// every row (136 terms, four rows of 5 10^4 samples 33 and 39, 16 of 10^5 104 and
// 138), so one pass stays there unless it spills: up to the real adjoint's one-pass
// size it runs at two waves per SIMD, whose registers more than 80 values of group
// sums and denominators overflow (64 terms, 106 values: 76 and 36 us, 323 and 130; 112
// terms, 104 values: 63 and 37, 235 and 132; 52 terms, 52 values: 24 and 27, 53 and 91).
constexpr int kJitAutoComplexBlockTerms = 200;
constexpr int kJitAutoComplexBlockTermsOneRow = 50;
// whether it does with this many rows, where the solution splits over the waves
bool jit_prefers_complex_block(const AmiTerms *t, bool one_row);

// Whether AUTO's adjoint of a solution up to kJitAutoAdjointTerms terms takes the
// block kernel: the one-pass kernel keeps a leaf and four values per group and
// denominator, and two per energy, live at once; beyond 100 of the 128 doubles
// that two waves per SIMD have, it spills (76 terms in 16 groups, 123 values,
// 2 10^5 samples: 58 us a step, the block kernel 40; 40 terms in 8 groups, 81
// values: 28 and 30; 52 terms in 4 groups, 68 values: 25 and 33).
bool jit_prefers_block_adjoint(const AmiTerms *t);

// Whether the adjoint of a solution above kJitAutoAdjointTerms can run in
// passes (the two-pass form, no Taylor-coefficient leaves).
bool jit_adjoint_passes_supported(const AmiTerms *t, bool hub, std::string *why);

// Waves per block of the block adjoint for this input, 0 when the solution has
// none (Taylor-coefficient leaves, too few groups to split evenly, or more
// columns than the LDS of a CU holds).  Chosen once per handle and input: the
// source and every launch of a handle take the same count, whatever becomes of the
// environment's override in between.  several: of the kernel for several frequency
// rows, where that is one of its own (jit_block_rows_apart).
int jit_block_waves(const AmiTerms *t, bool hub, bool cplx = false, bool several = false);
// Whether the real block adjoint has a kernel for one frequency row
// (kJitBlockAdjoint) and another for several (kJitBlockAdjointRows), else one for both.
bool jit_block_rows_apart(const AmiTerms *t);
int jit_block_forward_waves(const AmiTerms *t);   // of the block forward, 0: none

// Whether the diagram can be specialized for the energy (hub = false) or
// momentum (hub = true) input; *why says why not.
bool jit_supported(const AmiTerms *t, bool hub, std::string *why, bool two_pass = false);

// Whether AUTO evaluates the forward in two passes: the group sums and the
// reciprocals the one-pass kernel holds in registers across its frequency
// loop would exceed about half of a wave's registers.
bool jit_prefers_two_pass(const AmiTerms *t);

// Lanes per block of the specialized kernels.
int jit_block(const AmiTerms *t, bool hub);

// Device source of the specialized kernels: the forward (kernels & 1), the
// adjoint (kernels & 2), the Monte-Carlo integrator (kernels & 4), the
// forward at complex energies (kernels & 8), the two passes of the
// two-pass forward (kernels & 16: group sums and energies stored per sample;
// kernels & 32: per frequency, reciprocals and group products against them),
// and the passes of the adjoint of large solutions that follow the first of
// those (kernels & 64: per frequency, the group-sum and denominator
// cotangents; kernels & 128: the leaf cotangents and the gradients), the
// adjoint at complex energies (kernels & 256), and the two passes of the
// forward at complex energies (kernels & 512: complex group sums and energies
// stored per sample; kernels & 1024: per frequency, against them), and the
// passes of the adjoint at complex energies that follow the first of those
// (kernels & 2048: per frequency, the complex group-sum and denominator
// cotangents; kernels & 4096: the complex leaf cotangents and the gradients),
// and the block adjoint (kernels & 8192; its kernel for several frequency rows, where
// that is apart, 65536; at complex energies 16384) or the block
// forward (32768), each alone.
// nested_part: terms per part of the one-pass adjoint's leaf cotangents as a
// reverse sweep of the nested group sums (0: per-term prefix/suffix products;
// -1: the AMIGPU_JIT_NESTED_COTANGENTS override, else per-term products).
std::string jit_source(const AmiTerms *t, bool hub, int kernels, int nested_part = -1);

// The part size named by AMIGPU_JIT_NESTED_COTANGENTS, or -1.
int jit_nested_override();

// Terms per part of the nested leaf-cotangent sweep the one-pass adjoint
// tries beside the per-term products (the code object kept is chosen from
// the two compiled ones' registers and spills).
constexpr int kJitNestedPartTerms = 4;

// Unsigned ints between two work-list counters of a persistent batch kernel
// (one 128-byte cache line each).
constexpr int kBatchCounterStride = 32;

// Source of one module of the persistent specialized batch: the generated
// functions of every item (forward in one pass, or the two-pass forward where
// two_pass[j] is set; one_row[j]: the one-pass tile for exactly one frequency
// row) in a namespace of its own with the tile functions, all at `block`
// lanes per block, and the persistent kernels selected by `phases`:
// ami_batch_p1 (phases & 1: one-pass tiles and the two-pass items' first
// pass) and ami_batch_p2 (phases & 2, with any two-pass item: their frequency
// pass, a work item being a tile range at a range of rows).  The kernels take
// eight counters kBatchCounterStride apart, one per work list.
// A work item names its item by labels[j] (by j when labels is empty).
// claim_ahead: a block claims its next work item before it runs the current
// one (the claim's round trip overlaps the work, for a register more);
// waves > 0: the kernels are compiled for at least that many waves per SIMD.
std::string jit_batch_source(const std::vector<const AmiTerms *> &items, const std::vector<int> &two_pass,
                             const std::vector<int> &one_row, bool hub, int block, int phases,
                             const std::vector<int> &labels, bool claim_ahead = true, int waves = 0);

// An unsigned value of the kernel metadata of a code object built here (the
// integer after the key in its one kernel's note), or -1.
int64_t code_meta(const std::vector<char> &code, const char *key);

// Kernels of the specialized evaluator.
// kJitAdjFreq and kJitAdjLeaf are the frequency and leaf passes of the
// adjoint of large solutions (after kJitSumsPass); kJitComplexAdj is the
// adjoint at complex energies (energy input only, as kJitComplex);
// kJitComplexSums and kJitComplexFreq the two passes of the forward at complex
// energies (solutions above kJitMaxTerms terms); kJitComplexAdjFreq and
// kJitComplexAdjLeaf the frequency and leaf passes of the adjoint at complex
// energies (after kJitComplexSums); kJitBlockAdjoint the adjoint of large
// solutions whose work the waves of a block split (no workspace),
// kJitComplexBlockAdjoint the same at complex energies, kJitBlockForward the
// forward of large solutions that way, kJitBlockAdjointRows the block adjoint for
// several frequency rows where that is a kernel of its own.
enum JitKind {
    kJitForward = 0,
    kJitAdjoint = 1,
    kJitMonteCarlo = 2,
    kJitComplex = 3,
    kJitSumsPass = 4,
    kJitFreqPass = 5,
    kJitAdjFreq = 6,
    kJitAdjLeaf = 7,
    kJitComplexAdj = 8,
    kJitComplexSums = 9,
    kJitComplexFreq = 10,
    kJitComplexAdjFreq = 11,
    kJitComplexAdjLeaf = 12,
    kJitBlockAdjoint = 13,
    kJitComplexBlockAdjoint = 14,
    kJitBlockForward = 15,
    kJitBlockAdjointRows = 16
};
constexpr int kJitKinds = 17;

// Kinds for the energy input only (complex energies).
inline bool jit_kind_complex(int kind) {
    return kind == kJitComplex || kind == kJitComplexAdj || kind == kJitComplexSums || kind == kJitComplexFreq ||
           kind == kJitComplexAdjFreq || kind == kJitComplexAdjLeaf || kind == kJitComplexBlockAdjoint;
}

// The specialized kernel of `kind` for the energy (hub = false) or momentum
// input as a hipFunction_t: compiled (or fetched from the code-object cache)
// and loaded on the current device on first use; thread-safe per handle.
// The Monte-Carlo kernel exists for the momentum input only, the complex one
// for the energy input only.
AmiStatus jit_get(AmiTerms *t, bool hub, int kind, void **fn);

// Whether any device holds this kernel of the handle.
bool jit_has_module(AmiTerms *t, bool hub, int kind);

// jit_get for every device that holds a kernel of the handle for this input
// (the current device stays as it is).
AmiStatus jit_load_everywhere(AmiTerms *t, bool hub, int kind);

// The kernel of `kind` only if jit_get has already loaded it on the current
// device (loads nothing, allocates nothing): AMI_E_UNSUPPORTED when its
// compilation failed, AMI_E_ARG when it has not been loaded yet.
AmiStatus jit_loaded(AmiTerms *t, bool hub, int kind, void **fn);

// Only the code object of `kind` (compiled or fetched from the cache): needs
// no device.
AmiStatus jit_compile(AmiTerms *t, bool hub, int kind);

// The code object of a generated source: from the disk cache, else compiled
// with hipRTC under the library's flags and stored there.  Needs no device;
// thread-safe.  On failure err says why (the status is AMI_E_HIP).
AmiStatus code_from_source(const std::string &src, std::vector<char> &code, std::string &err);

// Unload every module of the handle (amiFree).
void jit_release(AmiTerms *t);

}  // namespace ami

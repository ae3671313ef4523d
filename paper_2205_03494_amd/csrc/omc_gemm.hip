// omc_dequant_gemm: C = A * decompress(W) with the weights expanded on chip (paper Sec. 2.1, forward path: the layer's
// parameters are decompressed on the fly and consumed at once), and omc_dequant_gemm_dx: dX = dY * decompress(W)^T.
//
// The affine per-variable transformation (Sec. 2.3) factors out of the contraction:
//     A (s Vt + b 1 1^T) = s (A Vt) + b rowsum(A) 1^T,
// and every code value Vt of a format with at most 7 mantissa bits is exactly a bfloat16, so the matrix cores run on exact
// images of the codes: bf16 x bf16 with fp32 accumulation.
#include "omc_gemm_bits_impl.h"

namespace omc {

// Host only, not part of the interface: index of the tile that a product of these sizes takes (columns N of the result, contraction K), in
// the table of the FP8 kernel or of the other formats' kernel.
extern "C" int omc_internal_gemm_tile(int fp8, uint32_t M, uint32_t N, uint32_t K) { return fp8 ? gemm_fp8_tile(M, N, K) : gemm_bits_tile(M, N, K); }
// Host only, not part of the interface: into how many chains of fp32 sums, of teams and in a team, that product's contraction is dealt.
extern "C" uint32_t omc_internal_gemm_sums(int fp8, uint32_t M, uint32_t N, uint32_t K) { return fp8 ? gemm_fp8_sums(M, N, K) : gemm_bits_sums(M, N, K); }

// C[M x N] = A[M x K] * W (trans == 0, W packed as [K x N]) or A * W^T (trans != 0, W packed as [N x K])
int launch_dequant_gemm(const uint16_t *A, const void *codes, const FmtParams &fp, const float *sb, float *C,
                        uint32_t M, uint32_t N, uint32_t K, int trans, void *stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (fp.bits == 8 && fp.variant == 2) return launch_gemm_fp8(A, codes, sb, C, M, N, K, trans, st);   // S1E4M3, bias 7
    const BitsArgs ga{A, static_cast<const uint32_t *>(codes), sb, C, N, K, 0, 0, fp};
    if (fp.bits <= 5) return launch_gemm_bits_2_5(ga, M, trans, st);
    if (fp.bits <= 8) return launch_gemm_bits_6_8(ga, M, trans, st);
    if (fp.bits <= 11) return launch_gemm_bits_9_11(ga, M, trans, st);
    if (fp.bits <= 14) return launch_gemm_bits_12_14(ga, M, trans, st);
    return launch_gemm_bits_15_16(ga, M, trans, st);
}

}  // namespace omc

"""Products whose reduction is split over the wavefronts of a workgroup: the exchange of the shares' partial sums.

A workgroup per 32 x 32 block has two, four or eight wavefronts, by the k-steps and the number of blocks.  In blocks of 64 x 128
reductions of at most 2^15 - 1 terms are exchanged as 16-bit numbers, longer ones in fp32.  Sums of whole numbers are exact, so
the integers have to agree with a float32 product of the same signs (exact below 2^24), up to rows and filters whose sum is
the whole reduction, of either sign."""
import pytest
import torch

from paper_1804_02941_amd import binding as dab

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _signs(words, n):
    """int32 words [rows, W] -> +1/-1 floats [rows, n]."""
    bits = (words.unsqueeze(-1) >> torch.arange(32, device=DEV, dtype=torch.int32)) & 1
    return bits.reshape(words.shape[0], -1)[:, :n].float()


# (rows, terms, filters) by kernel and what its plan chose, which test_host_sanitizers.py checks on the CPU: shares of the
# reduction (s1 to s8) in tiles of 64 x 128 and how they are exchanged, wavefronts of a 32 x 32 block, stores of fp32 outputs
CASES = {
    "split s8 16-bit": [(2048, 32767, 641)],                # 2^15 - 1 terms are the last in 16 bits; a last filter tile of one
    "split s8 fp32": [(2048, 32768, 641)],
    "split s4 16-bit": [(2050, 4096, 1280), (2048, 2400, 1284)],
    "split s4 fp32": [(2049, 33000, 1285)],
    "split s2 16-bit": [(8192, 2400, 640), (8191, 2336, 515), (40000, 2368, 40)],      # a row short, a filter count that is no multiple of four
    "split s2 fp32": [(8190, 32800, 1023)],
    "split s1 alone": [(81920, 2400, 40), (16300, 2368, 515),
                       (2, 64, 18400001)],                  # rows so long that 64 of them take more than 32 bits of offset
    # the k-steps and numbers of blocks where the wavefronts of a block change, one and four words a load
    "block s8": [(19, 9216, 4096), (31, 2048, 64)],
    "block s4": [(33, 960, 70), (33, 1024, 33), (33, 1088, 40), (31, 1984, 64), (2, 33, 1), (9, 256, 65), (2048, 960, 100),
                 (2049, 960, 100), (2049, 768, 37), (2049, 1088, 100)],
    "block s2": [(70001, 320, 1)],
    # many rows, the mask panel in LDS: last filters alone, in twos and in threes, whole and part tiles; 16-byte stores of rows
    # of any length
    "direct plain": [(70001, 320, 125), (70001, 320, 126), (70001, 320, 127), (70001, 320, 129), (70001, 320, 130), (70001, 320, 131), (300001, 320, 1),
                     (2304167, 32, 233), (4227330, 32, 127)],          # 2^29 - 1 and 2^29 - 2 values: nothing lands on the last ones
    "direct through": [(70001, 320, 132), (100001, 320, 160)],
    "direct streamed": [(170001, 320, 160)],                # above 96 MB in rows of 128-byte lines
}


@pytest.mark.parametrize("B,K,F", [c for cases in CASES.values() for c in cases])
def test_sums_of_shares(B, K, F):
    g = torch.Generator(device=DEV)
    g.manual_seed(B + K + F)
    W, Fp = (K + 31) // 32, 64 * ((F + 63) // 64)
    A = torch.randint(-2**31, 2**31, (B, W), generator=g, device=DEV).to(torch.int32)
    E = torch.randint(-2**31, 2**31, (W, Fp), generator=g, device=DEV).to(torch.int32)
    A[::7] = -1                                            # every sign +1, and every sign -1
    A[1::7] = 0
    E[:, ::5] = -1                                         # the whole reduction belongs to one group, or to the other
    E[:, 1::5] = 0
    if K % 32:
        A[:, -1] &= (1 << (K % 32)) - 1
        E[-1, :] &= (1 << (K % 32)) - 1
    E[:, F:] = 0
    alpha = torch.rand(F, generator=g, device=DEV) + 0.1
    beta = -torch.rand(F, generator=g, device=DEV) - 0.1
    tau = torch.randn(F, generator=g, device=DEV)
    a = 2.0 * _signs(A, K) - 1.0
    ref = a @ _signs(E.t().contiguous(), K)[:F].t().contiguous()
    sA = a.sum(dim=1, keepdim=True)
    ws = torch.empty(max(dab.lib().dab_binfc_workspace_bytes(B, K, F), 1), dtype=torch.uint8, device=DEV)
    Y, s1 = dab.dab_binfc(A, E, alpha, beta, K, want_s1=True, ws=ws)
    assert torch.equal(s1, ref.to(torch.int32))
    y64 = alpha.double() * ref.double() + beta.double() * (sA.double() - ref.double())
    # two roundings of terms of at most (|alpha| + |beta|) K each, at 2^-24
    assert (Y.double() - y64).abs().max() <= 4 * 2.0**-24 * 2.2 * K
    plain = dab.dab_binfc(A, E, alpha, beta, K, ws=ws)     # without the integers: the four-filter stores
    assert torch.equal(plain, Y)
    bits = dab.dab_binfc_bits(A, E, alpha, beta, K, tau, ws=ws)
    assert torch.equal(bits.reshape(B, -1), dab.dab_pack_activations(Y, dab.DAB_LAYOUT_NHWC, tau).reshape(B, -1))

"""Which calls of moe_layer_ffn run as a joint launch, both sides of every line of the rule (the library's own answer, no GPU needed)."""
import ctypes as C

import pytest

from paper_2602_03495_amd import binding as B


def joint(masked, T, d, N, k, I, shared=None):
    ok = B.load_library().moe_ffn_joint_ok
    ok.restype = C.c_bool
    ss = C.byref(B.shape(T, d, shared[0], shared[0], shared[1])) if shared else None
    return ok(C.byref(B.shape(T, d, N, k, I)), ss, C.c_bool(masked))


@pytest.mark.parametrize("masked,T,d,N,k,I,want", [
    (False, 384, 2048, 128, 8, 768, True), (False, 383, 2048, 128, 8, 768, False),           # routed rows, all experts on
    (False, 896, 2048, 8, 8, 2944, True), (False, 895, 2048, 8, 8, 2944, False),             # 56 tiles of few experts
    (False, 3072, 2048, 56, 1, 1408, True), (False, 3072, 2048, 55, 1, 1408, False),         # as many experts
    (True, 1024, 2048, 64, 6, 1408, True), (True, 1023, 2048, 64, 6, 1408, False),           # routed rows under a mask
    (True, 1152, 2048, 128, 8, 768, True), (True, 1151, 2048, 128, 8, 768, False),           # 72 to an expert
    (True, 9216, 2048, 56, 1, 1408, True), (True, 9216, 2048, 55, 1, 1408, False),           # experts under a mask
    (False, 2048, 2048, 128, 2, 512, True), (False, 2048, 1920, 128, 2, 512, False),         # hidden size
    (False, 4096, 2048, 128, 2, 384, True), (False, 4096, 2048, 127, 2, 384, False),         # up items
    (True, 4608, 2048, 128, 8, 128, True), (True, 4607, 2048, 128, 8, 128, False),           # ... under a mask
    (False, 8192, 2048, 64, 8, 8064, True), (False, 8192, 2048, 64, 8, 8192, False),         # inner size of the long-K kernel
    (False, 1024, 2048, 64, 4, 2048, False), (False, 1025, 2048, 64, 4, 2048, True),         # K split: up to 64 MB of partial sums
])
def test_routed_experts_alone(masked, T, d, N, k, I, want):
    assert joint(masked, T, d, N, k, I) == want


@pytest.mark.parametrize("T,d,N,k,I,S,Is,want", [
    (17, 512, 16, 2, 256, 2, 256, True), (16, 512, 16, 2, 256, 2, 256, False),               # more than a decode batch
    (17, 2048, 60, 4, 1408, 1, 2816, True), (17, 2048, 60, 4, 1408, 1, 2944, False),         # longer than two routed ones: 129 tokens
    (129, 2048, 60, 4, 1408, 1, 4224, True), (128, 2048, 60, 4, 1408, 1, 4224, False),
    (129, 2048, 60, 4, 1408, 1, 5632, True), (128, 2048, 60, 4, 4224, 1, 5632, False),       # a shared projection that splits K
    (2047, 1024, 60, 4, 1408, 1, 5632, False), (2048, 1024, 60, 4, 1408, 1, 5632, True),     # ... of a narrow layer
    (512, 2048, 64, 6, 1408, 1, 8064, True), (512, 2048, 64, 6, 1408, 1, 8192, False),
    (512, 2048, 64, 6, 8192, 1, 1408, False), (300, 2048, 8, 2, 2048, 1, 2048, False),       # routed: long K, K split
])
def test_with_shared_experts(T, d, N, k, I, S, Is, want):
    for masked in (False, True):
        assert joint(masked, T, d, N, k, I, (S, Is)) == want

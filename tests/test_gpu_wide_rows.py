"""bf16 GEMMs whose rows are too long for the LDS-DMA kernels' 32-bit offsets (from
2^22 elements on): the out-projection and dh of a block with an FFN of that
width, on the register-staged kernel, against the oracle.  The contraction is
no multiple of the kernel's K-tile either."""
import pytest

from paper_2402_15627_amd.inputs import BlockShape
from tests.parity_util import TOL, compare, case, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def test_ffn_of_four_million():
    s = BlockShape("wide", 1, 5, 8, 1, 64, (1 << 22) + 8, 3, "bf16")
    assert s.k_out % 64 == 8 and 256 * s.k_out * 2 >= 1 << 31
    print(f"[gpu] wide rows {s}", flush=True)
    inp = case(s, seed=1)
    errs, bad = compare(s, run_gpu(s, inp), run_oracle(s, inp))
    print("      " + ", ".join(f"{k}={v:.2e}" for k, v in errs.items()), flush=True)
    assert not bad, f"over tolerance {TOL['bf16']}: {bad}"

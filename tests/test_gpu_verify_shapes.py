"""The verify products' work splits and the attention's splits at their edges
(needs an MI355X with 256 CUs).  QKV is k_vpair with np = pairs / 256 row
pairs per workgroup, rounded up, and behind up to 256 visible positions the next
power of two, at most 32; gate/up is k_vgemm_sk there and k_vpair beyond.  Each case is
held to the bounds of the verify's oracle comparison: fp32 sums in another order,
and one bf16 rounding per cache entry."""
import pytest

from tests import test_gpu_verify as verify

pytestmark = pytest.mark.gpu

SHORT = dict(n_layers=1)
ONE = dict(n_layers=1, prompt_len=256)
WIDE_QKV = dict(n_layers=1, n_heads=64, n_kv_heads=64, head_dim=128)

CASES = {
    # gate/up with np pairs of rows per workgroup; the last workgroup is
    # ragged where np does not divide the pairs
    "np1": dict(ONE, ffn_dim=64),
    "np8": dict(ONE, ffn_dim=2048),
    "np9": dict(ONE, ffn_dim=2112),
    "np17": dict(ONE, ffn_dim=4160),
    "np25": dict(ONE, ffn_dim=6208),
    "np33": dict(ONE, ffn_dim=8256),
    "np49": dict(ONE, ffn_dim=12352),
    "np64": dict(ONE, ffn_dim=16384),
    # two rounds of workgroups, 33 pairs each
    "two_rounds": dict(ONE, ffn_dim=16448),
    "int8_np16": dict(ONE, ffn_dim=4096, wfmt="int8"),
    "int8_np17": dict(ONE, ffn_dim=4160, wfmt="int8"),
    "int8_np33": dict(ONE, ffn_dim=8256, wfmt="int8"),
    "int8_np49": dict(ONE, ffn_dim=12352, wfmt="int8"),
    # QKV of 12288 pairs, three ragged K stages: behind a short cache 384 workgroups
    # of 32 (half a head each), then 256 of 48 (which start inside a head and span
    # q, k and v)
    "qkv32": dict(WIDE_QKV, d_model=576),
    "qkv32_int8": dict(WIDE_QKV, d_model=576, wfmt="int8"),
    "qkv48": dict(WIDE_QKV, d_model=576, prompt_len=256),
    "qkv48_int8": dict(WIDE_QKV, d_model=576, prompt_len=256, wfmt="int8"),
    # gate/up ranges: 10 over two tile pairs of 16 stages, so that up to five meet
    # in one; 129 of two whole pairs; 256 of 2 or 3 units, ragged stages
    "sk_shared": dict(SHORT, d_model=4096, ffn_dim=64),
    "sk_shared_int8": dict(SHORT, d_model=4096, ffn_dim=64, wfmt="int8"),
    "sk_whole": dict(SHORT, ffn_dim=8256),
    "sk_ragged": dict(SHORT, d_model=576, ffn_dim=5568),
    # attention: one split of 8 blocks, the first of two splits, the merge of
    # nine splits (past eight it takes a wave per row)
    "splits1": dict(SHORT, prompt_len=246),
    "splits2": dict(SHORT, prompt_len=256),
    "splits9": dict(SHORT, prompt_len=2048, max_ctx=2112),
    "splits9_gqa_hd128": dict(SHORT, n_heads=4, n_kv_heads=1, head_dim=128, prompt_len=2048,
                              max_ctx=2112),
}


@pytest.mark.parametrize("name", list(CASES))
def test_verify_shapes(name, monkeypatch):
    monkeypatch.setitem(verify.CASES, name, CASES[name])
    verify.test_verify_equals_sequential_decode(name)

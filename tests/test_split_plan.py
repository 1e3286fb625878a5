"""Which layer steps a pass shares between groups of workgroups (split-K): the host's rule, on 256 CUs."""

import pytest

import workloads
from paper_2309_04255_amd import binding

# model, nodes: workgroups per group of QKV, O and down (gate/up is never shared)
RULE = [
    # up to 32 rows: none; 64 rows: the down projection in pairs; 4-bit: none
    ("llama7b", 31, 1, 1, 1), ("llama30b", 8, 1, 1, 1), ("llama7b_q4", 31, 1, 1, 1),
    ("llama7b", 33, 1, 1, 2), ("llama7b", 64, 1, 1, 2), ("llama13b", 41, 1, 1, 2), ("llama7b_q4", 64, 1, 1, 1),
    # 128 rows: O and down in fours; QKV in pairs only where a workgroup has more blocks than a
    # K-split tile holds (4): the 30B shape's 4.9, not the 13B's 3.75, the 7B's 3 or the 1B's 1.5
    ("llama7b", 65, 1, 4, 4), ("llama7b", 77, 1, 4, 4), ("llama7b", 128, 1, 4, 4), ("draft1b", 128, 1, 4, 4),
    ("llama13b", 77, 1, 4, 4), ("llama13b", 128, 1, 4, 4), ("llama30b", 77, 2, 4, 4), ("llama30b", 128, 2, 4, 4),
    # 4-bit: O and down in pairs
    ("llama7b_q4", 65, 1, 2, 2), ("llama7b_q4", 128, 1, 2, 2),
    # models without a block per group: none
    ("tiny", 128, 1, 1, 1), ("q4small", 128, 1, 1, 1),
]
SHAPES = workloads.MODELS


@pytest.fixture(autouse=True)
def defaults(monkeypatch):
    for k in ("PASS_GRID", "ROW_TILES", "SPLIT_QKV", "SPLIT_O", "SPLIT_DOWN"):
        monkeypatch.delenv(f"LLMCAD_{k}", raising=False)
    # (the same 256 workgroups on a host with another GPU)
    monkeypatch.setenv("LLMCAD_PASS_GRID", "256")


@pytest.mark.parametrize("model,n,qkv,o,down", RULE)
def test_rule(model, n, qkv, o, down):
    plan = binding.split_plan(binding.make_config(SHAPES[model]), n)
    assert {k: v[0] for k, v in plan.items()} == {"qkv": qkv, "o": o, "gate_up": 1, "down": down}
    for groups, rows, _ in plan.values():
        assert rows == (groups > 1 and n > 64)  # row-split or 4-bit tiles at 128 rows


def test_without_row_tiles(monkeypatch):
    # (diagnostics) 128-row passes then share as 64-row ones do
    monkeypatch.setenv("LLMCAD_ROW_TILES", "2")
    plan = binding.split_plan(binding.make_config(SHAPES["llama7b"]), 128)
    assert plan == {"qkv": (1, False, 3), "o": (1, False, 1), "gate_up": (1, False, 6), "down": (2, False, 2)}


@pytest.mark.parametrize("grid", [256, 200, 96, 64, 24, 8, 3])
@pytest.mark.parametrize("want", ["1", "2", "4", "8"])
@pytest.mark.parametrize("model", ["tiny", "q4small", "llama7b", "llama7b_q4", "llama30b"])
def test_groups_hold(monkeypatch, model, want, grid):
    # Whatever is asked for: whole groups with a block each, of a size that a tile takes.
    monkeypatch.setenv("LLMCAD_PASS_GRID", str(grid))
    for step in ("QKV", "O", "DOWN"):
        monkeypatch.setenv(f"LLMCAD_SPLIT_{step}", want)
    shape = SHAPES[model]
    blocks = {"qkv": 3 * shape.d_model // 16, "o": shape.d_model // 16, "down": shape.d_model // 16}
    for n in (31, 48, 64, 96, 128):
        plan = binding.split_plan(binding.make_config(shape), n)
        assert plan["gate_up"][0] == 1
        for step, nb in blocks.items():
            S, rows, largest = plan[step]
            assert S in (1, 2, 4) and (want in "124" or S == 1)
            if S > 1:
                assert grid % S == 0 and nb >= grid // S and largest == -(-nb // (grid // S))
            if rows:
                assert S > 1 and n > 64 and largest <= (6 if shape.weight_bits == 4 else 12)


def test_arguments():
    cfg = binding.make_config(SHAPES["tiny"])
    for n in (0, 129):
        with pytest.raises(binding.LlmcadError):
            binding.split_plan(cfg, n)
    assert binding.lib().llmcad_split_plan(cfg, 1, None) == binding.EARG

"""The shipped tuning cache holds the kinds that a kernel reads, and a cache
of earlier versions, with the inner products' range tiles, still loads."""
import json

from paper_2203_06233_amd import stap, tune


def test_shipped_cache_holds_what_is_read():
    kinds = {k.split("|")[1] for k in tune.load_cache()}
    assert kinds <= {"fused", "stage", "cov"} and "fused" in kinds


def test_earlier_cache_loads(tmp_path):
    saved = stap.tune_get(96, 32, "bf16", 1, kind=3)
    path = tmp_path / "cache.json"
    path.write_text(json.dumps({"gfx950|inner|dof<=96|s<=32|bf16|refine=1": {"variant": 2}}))
    try:
        assert tune.apply_cache(stap, str(path)) == 1
        assert stap.tune_get(96, 32, "bf16", 1, kind=3) == 2
    finally:
        stap.tune_set(96, 32, "bf16", 1, saved, kind=3)

"""The native calls of the Python binding: argument names, defaults and argument errors (no GPU needed)."""
import inspect

import pytest

import paper_2509_00419_amd as lv

CALLS = {
    "score_tokens": (["q", "k"], {"q_pos0", "img_begin", "n_img"}, {"scale": None, "causal": True, "row_lse": None,
                     "score_head": None, "score_mean": None, "reserve": True}),
    "score_from_probs": (["probs"], {"n_kv_heads", "img_begin", "n_img"}, {"score_head": None, "score_mean": None,
                         "reserve": True}),
    "prefill_attn": (["q", "k", "v"], set(), {"scale": None, "causal": True, "n_text": 0, "img_begin": 0, "n_img": 0,
                     "out": None, "row_lse": None, "score_head": None, "score_mean": None, "reserve": True}),
    "merge_compact": (["planes", "score_mean"], {"img_begin", "n_img", "n_keep"}, {"w": None, "rules": None, "outs": None,
                      "keep_idx": None, "merged_idx": None, "reserve": True}),
    "merge_similar": (["planes", "score_mean"], {"img_begin", "n_img", "n_keep"}, {"size": None, "rules": None, "outs": None,
                      "size_out": None, "keep_idx": None, "assign": None, "reserve": True}),
    "kv_compress": (["k_cache", "v_cache", "score", "kind", "orig_pos", "length"], {"mode"}, {"order": lv.ORDER_STABLE,
                    "beta": 0.995, "budget": 0, "n_recent": 0, "len_bound": 0, "n_evicted": None, "reserve": True,
                    "want_evicted": True}),
    "decode_attn": (["q", "k_new", "v_new", "k_cache", "v_cache", "score", "kind", "orig_pos", "length"], set(),
                    {"scale": None, "score_decay": 1.0, "new_kind": lv.KIND_GENERATED, "new_pos": 0, "len_bound": 0,
                     "evict_budget": 0, "evict_recent": 0, "out": None, "reserve": True, "static_scratch": False}),
}


@pytest.mark.parametrize("name", sorted(CALLS))
def test_native_calls_keep_their_arguments_and_refuse_others(name):
    positional, required, defaults = CALLS[name]
    pars = dict(inspect.signature(getattr(lv.Context, name)).parameters)
    pars.pop("self")
    assert [n for n, p in pars.items() if p.kind is p.POSITIONAL_OR_KEYWORD] == positional
    assert {n for n, p in pars.items() if p.kind is p.KEYWORD_ONLY and p.default is p.empty} == required
    assert {n: p.default for n, p in pars.items() if p.default is not p.empty} == defaults
    call, none = getattr(lv.Context(0), name), [None] * len(positional)
    full = dict.fromkeys(required, 1)
    for args, kw in (([], {}), (none[1:], full), (none + [None], full), (none, {**full, "nonsense": 1}),
                     (none, {**full, positional[0]: None}), (none, full)):
        with pytest.raises(TypeError):
            call(*args, **kw)

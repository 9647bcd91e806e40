"""The binding's descriptor: made once per strategy, kept out of what a
strategy is (equality, copies, pickles, field tables)."""

import copy
import dataclasses
import pickle

import paper_1710_08332_amd as dp


def test_descriptor_is_made_once_and_not_part_of_the_strategy():
    s = dp.Strategy(seq_len=16, local_size=64, order=dp.STRIDED, passes=1)
    fresh = dataclasses.replace(s)
    n = 16 * 64 * 5
    assert dp.strategy_check(s, dp.OP_DOT, dp.F32, 0, n) == \
        dp.strategy_check(fresh, dp.OP_DOT, dp.F32, 0, n)
    assert s._ref() is s._ref()
    assert s == dp.Strategy(seq_len=16, local_size=64, order=dp.STRIDED, passes=1)
    for t in (copy.copy(s), copy.deepcopy(s), pickle.loads(pickle.dumps(s)), s.with_(passes=2)):
        assert "_c" not in vars(t)
    assert pickle.loads(pickle.dumps(s)) == s
    assert set(dataclasses.asdict(s)) == {f.name for f in dataclasses.fields(dp.Strategy)}
    t = s.with_(seq_len=32)
    assert t._ref().contents.seq_len == 32 and s._ref().contents.seq_len == 16


def test_a_strategy_that_was_used_has_the_fields_of_one_that_was_not():
    s = dp.Strategy(seq_len=16, local_size=64, order=dp.STRIDED, passes=1)
    before = dict(vars(s))
    dp.strategy_check(s, dp.OP_DOT, dp.F32, 0, 4096)
    assert vars(s) == before
    assert dp.Strategy(**vars(s)) == s
    for t in (copy.copy(s), copy.deepcopy(s), pickle.loads(pickle.dumps(s))):
        assert t == s and vars(t) == before
        assert t._ref() is not s._ref()

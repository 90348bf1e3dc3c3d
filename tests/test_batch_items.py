"""Item shapes of the batched launch (host only): finer items and wide rollout tiles are taken where the estimate of an
instance's path says that they are shorter, never where they only add work."""
import ctypes

import pytest

import mtp_workloads as W
import paper_2505_01059_amd as mtp
from paper_2505_01059_amd import _native as N

UNITS = 256


def _contact24(total, horizon=256):
    return W.chain_contact_config(n_links=24, n_tensor=total - total // 17, n_gauss=total // 17, horizon=horizon,
                                  n_layers=12, n_width=64, n_elites=64, n_iters=2, ground_y=-4.0)


def _chain(links, total, horizon):
    return W.chain_config(n_links=links, n_tensor=total - total // 9, n_gauss=total // 9, horizon=horizon, n_layers=8,
                          n_width=32, n_elites=64, n_iters=3)


SETS = {
    "one large": [_contact24(69632)],
    "two large": [_contact24(69632)] * 2,
    "one share": [_contact24(8704)],
    "two shares": [_contact24(8704)] * 2,
    "four shares": [_contact24(8704)] * 4,
    "plain 24": [_chain(24, 16000, 128)],
    "two plain 24": [_chain(24, 16000, 128)] * 2,
    "four lanes of 4 links": [_chain(4, 22000, 128)],
    "small": [_chain(24, 1000, 64)],
    "mixed": [_contact24(8704), _chain(12, 3376, 64), _chain(7, 9216, 128)],
    "fleet of 4": [W.mix_instance(10000 + i) for i in range(4)],
    "fleet of 24": [W.mix_instance(10000 + i) for i in range(24)],
    "mix of 32": [W.mix_instance(i) for i in range(32)],
}


@pytest.mark.parametrize("name", SETS)
def test_no_instance_takes_a_longer_path(name):
    for it in mtp.batch_item_shapes(SETS[name], UNITS):
        assert it["path_us"] <= it["plain_path_us"] * (1 + 1e-12), it


@pytest.mark.parametrize("name,wide_lg", [("one large", 0), ("one share", 1), ("plain 24", 1),
                                          ("four lanes of 4 links", 1), ("small", 2)])
def test_a_lone_instance_takes_its_shortest_path(name, wide_lg):
    (it,) = mtp.batch_item_shapes(SETS[name], UNITS)
    assert it["wide_lg"] == wide_lg, it


def test_two_large_instances_keep_the_work_down():
    for it in mtp.batch_item_shapes(SETS["two large"], UNITS):
        assert it["wide_lg"] == 0 and it["work_us"] <= 1.1 * it["plain_work_us"], it


def test_never_split_keeps_the_plain_shape():
    for cfgs in SETS.values():
        for it in mtp.batch_item_shapes(cfgs, UNITS, split_pct=0):
            assert it["finest"] == 0 and it["wide_lg"] == 0 and it["path_us"] == it["plain_path_us"]


@pytest.mark.parametrize("name", ["mixed", "fleet of 4", "fleet of 24", "mix of 32"])
def test_a_short_queue_takes_back_only_what_does_not_fit(name):
    cfgs = SETS[name]
    full = mtp.batch_item_shapes(cfgs, UNITS)
    need = sum(it["items"] for it in full)
    plain = sum(it["items"] for it in mtp.batch_item_shapes(cfgs, UNITS, queue_items=1))   # every instance plain
    split = [i for i, it in enumerate(full) if it["path_us"] < it["plain_path_us"]]
    assert plain < need and split
    assert mtp.batch_item_shapes(cfgs, UNITS, queue_items=need) == full
    for room in (need - 1, (need + plain) // 2, plain):
        got = mtp.batch_item_shapes(cfgs, UNITS, queue_items=room)
        assert sum(it["items"] for it in got) <= room
        kept = [i for i in split if got[i] == full[i]]
        assert len(kept) == (len(split) - 1 if room == need - 1 else len(kept))
        for i in range(len(cfgs)):
            assert got[i] == full[i] or got[i]["path_us"] == got[i]["plain_path_us"]
    assert kept == []


def test_bad_arguments_are_refused():
    lib = mtp.load()
    assert lib.mtp_batch_item_shapes(None, 1, UNITS, None, 0, None) == 1
    cfg, keep = mtp.config_struct(SETS["small"][0])
    s, out = N.mtp_batch_schedule(0, 1, 1, 1, 64, 100), N.mtp_batch_items()
    for n in (0, 65537):   # as many as a batch takes
        assert lib.mtp_batch_item_shapes(ctypes.byref(cfg), n, UNITS, ctypes.byref(s), 0, ctypes.byref(out)) == 1
    with pytest.raises(mtp.MtpError):
        mtp.batch_item_shapes(SETS["small"], 0)
    with pytest.raises(mtp.MtpError):
        mtp.batch_item_shapes(SETS["small"], UNITS, cand_tiles=3)

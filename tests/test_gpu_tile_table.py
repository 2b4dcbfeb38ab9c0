"""The committed conv tile table covers every conv layer of the benchmark
workloads at every batch bucket they serve: with the default tile choice (the
table, timing only what it lacks) a pass at each bucket times nothing, so no
request waits for tile tuning, and every table entry names a tile that is a
candidate of its layer's kernel family (an entry that is not would fall back
to timing and show up here)."""
import re

import pytest

import workloads as wl
from paper_2003_01538_amd import flexserve as fsb
from paper_2003_01538_amd.make_tile_table import KEYS, PLAN, TABLE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("wname,max_batch,buckets", PLAN, ids=[p[0] for p in PLAN])
def test_table_covers_every_bucket(monkeypatch, wname, max_batch, buckets):
    monkeypatch.setenv("FS_TUNE", "2")  # the default: the table, timing what it lacks
    w = wl.workload(wname)
    with fsb.Ensemble(w["models"], w["out_hw"], wl.IMAGENET_MEAN, wl.IMAGENET_STD, w["precision"],
                      max_batch=max_batch) as ens:
        for b in buckets:
            print(f"{wname}: bucket {b}", flush=True)
            ens.infer(list(wl.images_uniform(w["image_seed"], b, *w["in_hw"])), want_logits=False)
        log = fsb.fs_tuning_log(ens.handle)
    assert log == "", f"{wname}: layers without a usable table entry:\n{log[:2000]}"


def test_the_log_records_timing(monkeypatch):
    # the control: with every layer timed (FS_TUNE=1) the same pass fills the
    # log, so an empty log above means nothing was timed
    monkeypatch.setenv("FS_TUNE", "1")
    wname, max_batch, buckets = PLAN[1]
    w = wl.workload(wname)
    with fsb.Ensemble(w["models"], w["out_hw"], wl.IMAGENET_MEAN, wl.IMAGENET_STD, w["precision"],
                      max_batch=max_batch) as ens:
        ens.infer(list(wl.images_uniform(w["image_seed"], buckets[0], *w["in_hw"])), want_logits=False)
        log = fsb.fs_tuning_log(ens.handle)
    assert "choice bucket" in log


def test_retiming_times_the_table_tile_first(monkeypatch):
    # FS_TUNE=3 (how the table is re-timed): every layer is timed, and the
    # table's tile comes first, so another candidate must beat it by the
    # tuner's margin to replace it
    entries = {}
    for m in re.finditer(r'\{(\d+(?:, \d+){12}), "([^"]+)"\}', open(TABLE).read()):
        entries[tuple(int(x) for x in m.group(1).split(", "))] = m.group(2)
    monkeypatch.setenv("FS_TUNE", "3")
    wname, max_batch, buckets = PLAN[1]
    w = wl.workload(wname)
    with fsb.Ensemble(w["models"], w["out_hw"], wl.IMAGENET_MEAN, wl.IMAGENET_STD, w["precision"],
                      max_batch=max_batch) as ens:
        ens.infer(list(wl.images_uniform(w["image_seed"], 32, *w["in_hw"])), want_logits=False)
        log = fsb.fs_tuning_log(ens.handle)
    first, checked = {}, 0
    for line in log.splitlines():
        f = line.split()
        if line.startswith("bucket "):
            first.setdefault((f[3], f[5]), f[f.index("tile") + 1])
        elif line.startswith("choice "):
            kv = dict(zip(f[1::2], f[2::2]))
            key = tuple(int(kv[k]) for k in KEYS)
            if key in entries and (kv["group"], kv["layer"]) in first:
                assert first[(kv["group"], kv["layer"])] == entries[key], line
                checked += 1
    assert checked >= 10



def test_layers_that_run_in_one_launch_are_not_timed(monkeypatch):
    # one ResNet-50: from nine images on its 56 x 56 blocks' widening and narrowing
    # 1x1 convs always share a launch, so no batch of the 16-image bucket uses a
    # tile of theirs; in the 8-image bucket five images still do
    monkeypatch.setenv("FS_TUNE", "1")
    w = wl.workload("resnet50x5_bf16_b256")
    with fsb.Ensemble(w["models"][:1], w["out_hw"], wl.IMAGENET_MEAN, wl.IMAGENET_STD, w["precision"],
                      max_batch=16) as ens:
        timed = {}
        for b in (8, 16):
            imgs = list(wl.images_uniform(w["image_seed"], b, *w["in_hw"]))
            fsb.fs_profile_enable(ens.handle)
            ens.infer(imgs, want_logits=False)
            pairs = {l["layer"] for l in fsb.fs_profile_launches(ens.handle) if l["kernel"] == "conv_pair_1x1"}
            fsb.fs_profile_enable(ens.handle, False)
            log = fsb.fs_tuning_log(ens.handle)
            timed[b] = {int(m.group(1)) for m in re.finditer(rf"choice bucket {b} group 0 layer (\d+)", log)}
            assert pairs, b
            both = pairs | {i + 1 for i in pairs}
            assert both <= timed[b] if b == 8 else not both & timed[b], (b, both, timed[b])
        assert timed[8] - timed[16] == both


def test_ruled_tiles_follow_the_batch_and_not_its_bucket():
    # three ResNet-18s, 14 x 14 x 256: the tile for twelve images is not the one for sixteen
    w = wl.workload("resnet18x3_bf16_b32")
    with fsb.Ensemble(w["models"], w["out_hw"], wl.IMAGENET_MEAN, wl.IMAGENET_STD, w["precision"], max_batch=16) as ens:
        ran = {}
        for b in (12, 16):
            fsb.fs_profile_enable(ens.handle)
            ens.infer(list(wl.images_uniform(w["image_seed"], b, *w["in_hw"])), want_logits=False)
            ran[b] = {l["kernel"] for l in fsb.fs_profile_launches(ens.handle) if (l["N"], l["K"]) == (256, 2304)}
            fsb.fs_profile_enable(ens.handle, False)
            want = {fsb.fs_test_conv_choice(b, 14, 14, 256, 256, 3, 1, 1, fsb.FS_BF16, 3, residual=r)[0] for r in (0, 1)}
            assert ran[b] == want, b
        assert ran[12] != ran[16]

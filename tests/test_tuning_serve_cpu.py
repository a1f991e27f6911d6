"""The launch class of a server (no GPU): its own entry, else the batch's."""

from workloads import workload


def test_a_server_takes_its_own_class_or_the_batch():
    from paper_1202_2355_amd import tuning
    lay = workload(3).layout
    assert tuning.class_key("serve", "f32", lay) == "serve:f32:losvd"
    one = {"batch:f32:losvd": {"params": {"tiles_per_cu": 6}}}
    assert tuning.lookup("serve", "f32", lay, None, one)["tiles_per_cu"] == 6
    both = dict(one, **{"serve:f32:losvd": {"params": {"tiles_per_cu": 16, "groups": 1}}})
    assert tuning.lookup("serve", "f32", lay, None, both)["groups"] == 1
    assert tuning.lookup("batch", "f32", lay, None, both)["tiles_per_cu"] == 6
    assert tuning.lookup("serve", "f64", lay, None, both) == tuning.DEFAULT_F64
    # the stored table: one group, so that work beside the batch finds its turn
    assert tuning.lookup("serve", "f32", lay)["groups"] == 1

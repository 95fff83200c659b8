"""The tuning table of a network keeps which kernel each layer takes, however often it is written and read.  Needs no GPU."""
from paper_2011_06295_amd import harness, workloads as wl


def _kernels(net):
    return [r.layer.get_kernel(net.work.N, r.spec.H, r.spec.W, r.spec.stride, r.spec.pad) for r in net.runs]


def test_table_keeps_the_matrix_kernel(tmp_path):
    path = str(tmp_path / "table.json")
    work = wl.vgg16(256, "f16")
    net = harness.Network(work)
    kernels = _kernels(net)
    assert "matrix" in kernels and "tile" in kernels
    for _ in range(3):          # nothing tuned; then read, written, read and written again
        table = net.save_table(path)
        for li, kernel in enumerate(kernels):
            assert (table[net.table_key(li)]["launch"] == []) == (kernel == "matrix")
        net.close()
        net = harness.Network(work)
        assert net.load_table(path) == len(net.runs)
        assert _kernels(net) == kernels
    # a pinned launch stays pinned
    li = kernels.index("matrix")
    run = net.runs[li]
    pinned = run.layer.rank_launches(work.N, run.spec.H, run.spec.W, run.spec.stride, run.spec.pad, 1)[0]
    run.layer.set_launch(pinned)
    net.save_table(path)
    net.close()
    net = harness.Network(work)
    net.load_table(path)
    assert _kernels(net)[li] == "tile"
    net.close()

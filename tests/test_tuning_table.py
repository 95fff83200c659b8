"""The tuning table of a network keeps which kernel each layer takes, however often it is written and read.  Needs no GPU."""
from paper_2011_06295_amd import harness, workloads as wl


def _kernels(net):
    return [r.layer.get_kernel(net.work.N, r.spec.H, r.spec.W, r.spec.stride, r.spec.pad) for r in net.runs]


def test_table_keeps_the_matrix_kernel(tmp_path):
    path = str(tmp_path / "table.json")
    # (layers that are far from where the two kernels meet: 17 us are estimated for the matrix kernel and 11 for the other, 12 and 39)
    work = wl.Workload("two_kernels", 31, 64, "f16", "normal", [
        wl.LayerSpec("thin", C=512, K=512, R=3, S=3, H=2, W=2, pad=1, sparsity_bp=9900),
        wl.LayerSpec("thick", C=128, K=128, R=3, S=3, H=14, W=14, pad=1, sparsity_bp=7000)], chain=False)
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

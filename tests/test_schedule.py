"""Which kernels the library launches, on devices of made-up sizes: tests/fake_device.cpp stands in for the HIP runtime, so the
library's own host code decides and nothing runs.  No launch of workgroups that wait for one another may be larger than the
device, and a pass that no such kernel can take runs launch by launch."""
import math
import os
import random
import subprocess

import pytest

from paper_2001_04206_amd import build, dn

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def device(tmp_path_factory):
    if not os.path.exists(dn.LIB_PATH):
        build.build()
    exe = str(tmp_path_factory.mktemp("fake_device") / "fake_device")
    lib = os.path.dirname(dn.LIB_PATH)
    plans = exe + "_plans.o"
    subprocess.run([build.HIPCC, "-x", "hip", "--offload-host-only", "-fPIC", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(lib, "csrc"), "-c",
                    os.path.join(HERE, "fake_plans.cpp"), "-o", plans], check=True)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "include"), os.path.join(HERE, "fake_device.cpp"), plans, "-o", exe,
                    "-L" + lib, "-l:libdn.so", "-Wl,--export-dynamic,--allow-shlib-undefined,--disable-new-dtags,-rpath," + lib +
                    ",-rpath,/opt/rocm/lib"], check=True)

    def run(units, *commands, arguments=False, plans=False, names=False):
        """One (status, schedule, [(kernel, workgroups)]) per command; [(kernel, template arguments)] with arguments=True,
        [(kernel, what its parameters say)] with plans=True; the schedule's kernel (dn_last_kernel) in its place with names=True."""
        out = subprocess.run([exe, str(units), *commands], check=True, capture_output=True, text=True, timeout=120).stdout
        rows = []
        for line in out.splitlines():
            status, schedule, *launches = line.split()
            schedule, kernel = schedule.split("=")
            launches = [l.split("/") for l in launches]
            rows.append((int(status), kernel if names else int(schedule), [(l[0], l[3] if plans else l[2] if arguments else int(l[1])) for l in launches]))
        assert len(rows) == len(commands), out
        return rows

    return run


WAITING = ("online_epoch_kernel", "twin_epoch_kernel", "wide_epoch_kernel", "wide_block_epoch_kernel", "block_epoch_kernel", "batch_epoch_kernel",
           "deep_batch_epoch_kernel")
NETS = ["784-128-10:ce", "256-256-10:ce", "1024-1000-16:ce", "64-512-64:ce", "5-999-2:mse", "340-100000-10:ce", "340-38000-3:mse", "4-16-3:ce"]


@pytest.mark.parametrize("units", [256, 128, 36, 21, 8, 2, 1])
@pytest.mark.parametrize("net", NETS)
def test_batch_1_passes_on_devices_of_any_size(device, net, units):
    passes = ["train:96:1:0", "train:96:1:0.9", "train:63:1:0", "train:63:1:0.9", "option:online_blocks=0", "train:96:1:0"]
    for command, (status, schedule, launches) in zip(passes, device(units, "net:%s:1" % net, *passes)[1:]):
        assert status == dn.DN_OK, command
        for kernel, grid in launches:
            if kernel in WAITING:
                assert grid <= units, (command, kernel, grid)
        if command.startswith("train"):
            assert launches and schedule != dn.DN_SCHED_NONE


def test_digits_take_blocks_only_when_they_fit(device):
    for units, blocks in ((256, True), (37, True), (36, False)):
        rows = device(units, "net:784-128-10:ce:1", "train:64:1:0", "train:63:1:0", "train:64:1:0.5", "option:online_blocks=0", "train:64:1:0")
        assert [r[1] == dn.DN_SCHED_SAMPLE_BLOCKS for r in rows[1:]] == [blocks, False, False, False, False]
        if blocks:
            assert rows[1][2] == [("block_epoch_kernel", 37)]


def test_wide_hidden_layers_report_their_own_schedule(device):
    rows = device(256, "net:340-38000-3:ce:1", "train:64:1:0", "train:63:1:0", "train:64:1:0.5", "option:online_blocks=0", "train:64:1:0")
    assert [r[1] for r in rows[1:]] == [dn.DN_SCHED_WIDE_BLOCKS, dn.DN_SCHED_WIDE_HIDDEN, dn.DN_SCHED_WIDE_HIDDEN, dn.DN_SCHED_WIDE_HIDDEN,
                                        dn.DN_SCHED_WIDE_HIDDEN]
    assert dn.SCHEDULE_KERNELS[rows[1][1]] in [k for k, _ in rows[1][2]]
    # the kernel that sweeps W_1 every step: by itself, and in the form that looks whether it was left the samples
    rows = device(256, "net:340-38000-3:ce:1", "train:63:1:0", "train:64:1:0", arguments=True)
    assert [dict(r[2]).get("wide_epoch_kernel") for r in rows[1:]] == ["<12,false,false>", "<12,false,true>"]


def test_nets_of_one_wavefront_hold_no_blocks(device):
    """Every layer at most 64 wide: no room in the arena for inner products that nothing forms, whatever runs the passes."""
    products = 4096 // 32 * 2 * 32 * 32 * 8
    for widths in ([4, 16, 3], [64, 64, 64]):
        assert dn.dn_net_arena_bytes(widths, 1) < dn.dn_net_arena_bytes([65, 64, 64], 1) - products // 2
        rows = device(256, "net:%s:ce:1" % "-".join(map(str, widths)), "train:96:1:0", "option:online_tiny=0", "train:96:1:0")
        assert rows[1][1] == dn.DN_SCHED_ONE_WAVE_REGISTERS and rows[3][1] in (dn.DN_SCHED_ONE_WORKGROUP, dn.DN_SCHED_TWO_COPY), rows


# net, rows: whether dn_forward takes the last layer in one launch
@pytest.mark.parametrize("net,rows,one", [
    ("16-100000-10:ce", 1, False), ("16-100000-10:ce", 1024, False), ("16-16384-16:ce", 64, False), ("16-8193-4:ce", 1, False), ("16-8192-4:ce", 768, True),
    ("16-8192-4:ce", 769, False), ("1024-1024-10:ce", 2048, True), ("1024-1024-10:ce", 2049, False), ("16-1024-16:ce", 2048, True),
    ("16-1025-16:ce", 769, False), ("16-512-16:ce", 769, True), ("16-511-16:ce", 769, False), ("64-96-10:ce", 128, True), ("64-96-17:ce", 128, False),
    ("16-100000-10:mse", 1, False), ("16-1024-16:mse", 768, True), ("16-1024-16:mse", 769, False), ("16-1023-16:mse", 512, True),
    ("16-1023-16:mse", 513, False), ("16-512-11:mse", 512, True), ("16-511-11:mse", 1, False), ("16-256-10:mse", 64, True), ("16-255-3:mse", 64, False),
    ("16-1025-16:mse", 1, False), ("16-64-16:mse", 1, False)])
def test_narrow_last_layers_of_predictions(device, net, rows, one):
    status, _, launches = device(256, "net:%s:%d" % (net, rows), "forward:%d" % rows)[1]
    assert status == dn.DN_OK and ("narrow_output_kernel" in [k for k, _ in launches]) == one, launches


# rows, terms of a sum, outputs: the tile of the forward product on either side of the lines of the eight-wave tile
@pytest.mark.parametrize("rows,k,n,tile", [
    (330, 280, 1356, "32,64,8"), (222, 1472, 2112, "32,64,8"), (641, 1628, 768, "32,64,8"), (776, 4416, 640, "32,64,8"), (666, 619, 739, "32,32,8"),
    (513, 1000, 960, "32,64,8"), (512, 1000, 1024, "32,64,8"), (513, 1000, 1024, "64,64,8"), (1024, 1000, 1024, "64,64,8"), (1025, 1000, 1024, "64,64,4"),
    (128, 4544, 2048, "32,64,8"), (131, 4544, 1376, "32,64,8"), (609, 3552, 416, "64,64,8"), (609, 3068, 416, "32,64,8"), (1363, 3088, 320, "32,64,8"),
    (799, 4032, 544, "64,64,8"), (799, 3580, 544, "32,64,8"), (436, 3073, 999, "64,64,8"), (131, 4545, 1376, "64,64,8"), (298, 520, 1632, "32,32,8"), (395, 4512, 1248, "32,32,8"),
    (1163, 873, 418, "64,64,8")])
def test_tiles_of_forward_products(device, rows, k, n, tile):
    status, _, launches = device(256, "net:%d-%d:mse:%d" % (k, n, rows), "forward:%d" % rows, arguments=True)[1]
    products = [a for name, a in launches if name == "gemm_kernel"]
    assert status == dn.DN_OK and len(products) == 1 and products[0].startswith("<dn::SliceTile<%s," % tile), launches


# net, batch, momentum: whether a pass runs on the kernel that cuts every layer into tiles
@pytest.mark.parametrize("net,batch,mu,tiles", [
    ("784-128-10:ce", 128, 0.9, True), ("1024-1024-1024-1024-10:ce", 32, 0, True), ("1024-1024-1024-1024-10:ce", 64, 0, False), ("64-96-80-10:ce", 8, 0.9, True),
    ("300-500-200-300:ce", 33, 0.9, True), ("48-67-28:ce", 54, 0.9, False), ("1288-19-4:ce", 4, 0, False), ("123-10-55:ce", 147, 0, False),
    ("1024-1025-1024-10:ce", 16, 0, False), ("100-50-1024:ce", 8, 0, True), ("100-50-1025:ce", 8, 0, False), ("200-120-10:ce", 257, 0, False)])
def test_passes_on_tiles(device, net, batch, mu, tiles):
    for units in (256, 100, 8, 1):
        train = "train:%d:%d:%g" % (3 * batch, batch, mu)
        rows = device(units, "net:%s:%d" % (net, batch), train, "option:batch_tiles=0", train)
        assert all(r[0] == dn.DN_OK for r in rows)
        ran = [grid for kernel, grid in rows[1][2] if kernel == "tile_epoch_kernel"]
        assert all(grid <= units for grid in ran) and rows[1][2]
        if units == 256:
            assert bool(ran) == tiles, rows
        assert "tile_epoch_kernel" not in [k for k, _ in rows[3][2]]


# net, momentum: whether a batch-1 pass runs on as few workgroups as hold it, and on how many
@pytest.mark.parametrize("net,mu,groups", [
    ("37-116-21-61:ce", 0, 1), ("37-116-21-61:ce", 0.9, 1), ("96-64-160-440-37:ce", 0, 3), ("192-68-7:ce", 0.9, 1), ("192-68-7:ce", 0, None),
    ("1024-1024-1024-1024-10:ce", 0, None), ("28-16-32-188-19:ce", 0, 1), ("544-44-224-2:ce", 0, None), ("4-32-736-10:ce", 0, None), ("376-156-32-5:ce", 0, None),
    ("18-10-21-7-23:ce", 0.9, None), ("14-24-4-36-15:ce", 0.9, 1), ("4-16-3:ce", 0.9, None), ("340-100000-10:ce", 0.9, None),
    ("20-30-20-30-20-5:ce", 0, None), ("100-70-60-129:ce", 0, None)])
def test_passes_on_few_workgroups(device, net, mu, groups):
    for units in (256, 8, 1):
        rows = device(units, "net:%s:1" % net, "train:32:1:%g" % mu, "option:online_slices=0", "train:32:1:%g" % mu, "option:online_mode=1",
                      "option:online_slices=2", "train:32:1:%g" % mu)
        assert all(r[0] == dn.DN_OK for r in rows), rows
        ran = [grid for kernel, grid in rows[1][2] if kernel == "slice_epoch_kernel"]
        assert all(grid <= units for grid in ran) and (rows[1][1] == dn.DN_SCHED_SLICES) == bool(ran)
        if units == 256:
            assert ran == ([] if groups is None else [groups if groups == 1 else 8 * groups]), rows
        assert not [1 for r in (rows[3], rows[6]) for kernel, _ in r[2] if kernel == "slice_epoch_kernel"]


def test_workgroups_that_wait_are_waited_for(device):
    """A workgroup of the few that hold a net has units of some hidden layer, or nobody would wait for it and its words would be
    overwritten before it reads them."""
    rng = random.Random(4)
    width = lambda: int(math.exp(rng.uniform(math.log(2), math.log(2049))))
    nets = ["1000-1000-33:ce", "868-544-896-640-3:ce", "900-805-210-3:ce", "920-873-8:ce", "768-704-28-10:ce", "2048-85-4:ce"]
    nets += ["%s-%d:ce" % ("-".join(str(width()) for _ in range(rng.choice([2, 3, 4]))), rng.randint(1, 128)) for _ in range(120)]
    took = 0
    for units in (256, 32):
        commands = [c for net in nets for c in ("net:%s:1" % net, "option:online_slices=2", "train:32:1:0", "train:32:1:0.9")]
        for status, _, launches in device(units, *commands, plans=True):
            assert status == dn.DN_OK
            for kernel, plan in launches:
                if kernel == "slice_epoch_kernel":
                    groups, owning = map(int, plan.split("of"))
                    assert groups == owning
                    took += groups > 1
    assert took > 100


def test_layers_on_eight_images_a_lane(device):
    """The layers by which tests/test_gpu_conv_dw.py tests conv_dw_images_kernel are ones that take it; narrow or padded ones do not."""
    from test_gpu_conv_dw import LONG, ODD, SHAPES
    others = [(8, 8, 14, 14, 32, 1), (256, 16, 64, 64, 32, 1), (57, 31, 30, 30, 63, 0)]
    shapes = SHAPES + [LONG, ODD] + others
    rows = device(256, *["convback:%d:%d:%d:%d:%d:3:1:%d" % s for s in shapes], "convback:128:32:32:32:64:5:1:2", "convback:128:32:32:32:64:3:2:1")
    assert all(r[0] == dn.DN_OK for r in rows)
    took = ["conv_dw_images_kernel" in [k for k, _ in r[2]] for r in rows]
    assert took == [True] * (len(SHAPES) + 2) + [False] * (len(others) + 2)


# net, largest batch, pass, options: every schedule
PASSES = [("4-16-3:ce", 1, "64:1:0", ()), ("4-16-3:ce", 1, "64:1:0.9", ()), ("784-128-10:ce", 1, "64:1:0", ()), ("784-128-10:ce", 1, "63:1:0", ()),
          ("1024-1024-1024-1024-10:ce", 1, "8:1:0", ()), ("1024-1024-1024-1024-10:ce", 1, "8:1:0.9", ("online_slices=0",)),
          ("37-116-21-61:ce", 1, "8:1:0", ()), ("340-100000-10:ce", 1, "63:1:0", ()), ("340-100000-10:ce", 1, "64:1:0", ()),
          ("784-128-10:ce", 128, "256:128:0.9", ()), ("784-128-10:ce", 128, "256:128:0.9", ("batch_tiles=0",)), ("784-512-10:ce", 64, "128:64:0.9", ()),
          ("784-512-10:ce", 64, "128:64:0.9", ("batch_tiles=2",)), ("1024-1024-1024-1024-10:ce", 8, "16:8:0", ("batch_mode=2",)),
          ("1024-1024-1024-1024-10:ce", 32, "64:32:0", ()), ("4096-4096-4096-1000:ce", 256, "512:256:0.9", ()), ("784-128-10:ce", 1, "8:1:0", ("online_mode=1",))]


def test_the_kernel_of_a_pass_is_known_by_name(device):
    """dn_last_kernel names a kernel that the pass launched, and none where it went launch by launch."""
    seen = set()
    for net, batch, run, options in PASSES:
        commands = ["net:%s:%d" % (net, batch)] + ["option:" + o for o in options] + ["train:" + run]
        schedule, kernel = device(256, *commands)[-1][1], device(256, *commands, names=True)[-1][1]
        launched = [k for k, _ in device(256, *commands)[-1][2]]
        assert kernel in launched if kernel else schedule == dn.DN_SCHED_LAUNCHES, (net, options, kernel, launched)
        assert kernel in ("", "tile_epoch_kernel", dn.SCHEDULE_KERNELS.get(schedule)), (net, kernel)
        seen.add((schedule, kernel))
    assert len(seen) == 14
    assert device(256, "net:4-16-3:ce:1", names=True)[0][1] == ""


@pytest.mark.parametrize("net,batch,after", [("200-120-10:ce", 24, "batch_epoch_kernel"), ("64-96-80-100:ce", 24, None)])
def test_a_launch_of_tiles_that_is_kept_apart(device, net, batch, after):
    """The pass begins on tiles and ends on the schedule it has without them."""
    train = "train:%d:%d:0.9" % (4 * batch, batch)
    commands = ("net:%s:%d" % (net, batch), "option:batch_tiles=3", train, "option:batch_tiles=0", train)
    rows, plans = device(256, *commands), device(256, *commands, plans=True)
    assert all(r[0] == dn.DN_OK for r in rows)
    assert plans[2][2][0] == ("tile_epoch_kernel", "kept-apart") and rows[2][2][1:] == rows[4][2]
    assert rows[2][1] == rows[4][1] and (after is None or rows[2][2][1][0] == after)


def test_nets_by_which_tiles_are_tested(device):
    from test_gpu_tiles import CE, NETS
    for widths, _, loss, batch, n in NETS + [([12, 20, 3], 0, CE, 225, 500), ([30, 70], 0, CE, 257, 600)]:
        net = "net:%s:%s:%d" % ("-".join(map(str, widths)), "ce" if loss == CE else "mse", batch)
        took = device(256, net, "option:batch_tiles=2", "train:%d:%d:0.7" % (n, batch), names=True)[2][1] == "tile_epoch_kernel"
        assert took == (batch not in (225, 257)), (widths, batch)


def test_tiles_rest_after_a_launch_that_was_kept_apart(device):
    """8 passes, 16 after the next such launch, and so on; setting the option begins anew."""
    tried = lambda rows: ["tile_epoch_kernel" in [k for k, _ in r[2]] for r in rows]
    train = "train:96:24:0.9"
    rows = device(256, "net:200-120-10:ce:24", "option:batch_tiles=3", *[train] * 60, "option:batch_tiles=2", train, train)
    assert [i for i, t in enumerate(tried(rows[2:62])) if t] == [0, 9, 26, 59]
    assert tried(rows[-2:]) == [True, True]
    rows = device(256, "net:200-120-10:ce:24", "option:batch_tiles=3", *[train] * 2000)
    assert [i for i, t in enumerate(tried(rows[2:])) if t] == [0, 9, 26, 59, 124, 253, 510, 1023]


@pytest.mark.parametrize("net,mu", [("37-116-21-61:ce", 0), ("838-953-33-75-87:ce", 0.9), ("1000-1000-33:ce", 0.9), ("28-16-32-188-19:ce", 0), ("36-54-15-32:ce", 0)])
def test_options_of_the_general_kernel_leave_it_the_pass(device, net, mu):
    """"online_min_tile" and "online_resident" say how the kernels that own rows run: the few workgroups do not take the pass then."""
    train = "train:32:1:%g" % mu
    rows = device(256, "net:%s:1" % net, train, "option:online_min_tile=64", train, "option:online_min_tile=4096", train, "option:online_resident=0", train,
                  "option:online_slices=2", train, "option:online_slices=0", train, names=True)
    ran = [r[1] for r in rows if r[2]]
    assert [k == "slice_epoch_kernel" for k in ran] == [True, False, True, False, True, False] and ran[3] == ran[5]


# net, momentum, samples: passes of few samples, whose time is what a call costs, and nets whose steps the other kernel takes faster
@pytest.mark.parametrize("net,mu,n,few", [
    ("9-16-64-3:ce", 0, 1, False), ("9-16-64-3:ce", 0, 200, True), ("36-54-15-32:ce", 0, 1, False), ("36-54-15-32:ce", 0, 2, True),
    ("124-748-476-504-10:ce", 0, 1, False), ("124-748-476-504-10:ce", 0, 8, True), ("3-1322-410-38:ce", 0.9, 1, True), ("4-32-643-7:ce", 0, 4, False),
    ("40-8-1384-4:ce", 0, 40, False), ("4-932-16-8:ce", 0, 1, False), ("4-932-16-8:ce", 0, 40, True), ("16-832-3:ce", 0.9, 10000, False),
    ("192-68-7:ce", 0.9, 1, True), ("4-1952-3:ce", 0.9, 10000, False)])
def test_short_passes_stay_where_they_were(device, net, mu, n, few):
    row = device(256, "net:%s:1" % net, "train:%d:1:%g" % (n, mu))[1]
    assert row[0] == dn.DN_OK and (row[1] == dn.DN_SCHED_SLICES) == few, row


@pytest.mark.parametrize("net,batch,steps,tiles", [
    ("784-128-10:ce", 128, 1, False), ("784-128-10:ce", 128, 8, True), ("1024-1024-1024-1024-10:ce", 32, 1, True), ("16-21:ce", 234, 100, False),
    ("304-3:ce", 157, 100, False), ("12-3:ce", 19, 100, False), ("392-112:ce", 19, 4, True), ("24-888-4:ce", 43, 100, False), ("24-416-11:ce", 10, 4, True)])
def test_few_steps_and_narrow_nets_without_tiles(device, net, batch, steps, tiles):
    row = device(256, "net:%s:%d" % (net, batch), "train:%d:%d:0.9" % (steps * batch, batch), names=True)[1]
    assert row[0] == dn.DN_OK and (row[1] == "tile_epoch_kernel") == tiles, row


@pytest.mark.parametrize("units", [8, 32, 64])
def test_passes_that_waited_for_nobody_still_do_not(device, units):
    """A net that fits no kernel whose workgroups wait for one another but the few workgroups' one runs launch by launch; on one workgroup
    it may run there."""
    for net, mu in (("838-953-33-75-87:ce", 0.9), ("140-225-1480-3:ce", 0), ("567-79-8-1-63:ce", 0.9), ("37-116-21-61:ce", 0), ("192-68-7:ce", 0.9), ("128-96-40-10:ce", 0)):
        rows = device(units, "net:%s:1" % net, "train:8:1:%g" % mu, "option:online_slices=0", "train:8:1:%g" % mu)
        if rows[3][1] == dn.DN_SCHED_LAUNCHES:
            assert [k for k in rows[1][2] if k[0].endswith("epoch_kernel")] in ([], [("slice_epoch_kernel", 1)]), (net, rows[1])

"""The host engine's bookkeeping on a HIP runtime without a device: what it does when the
device has no room."""
import pytest

import fake_device


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    return fake_device.build(tmp_path_factory.mktemp("fake_device"))


def test_the_runtime_is_the_fake_one(fake):
    """(No other test here means anything otherwise.) Kernels' buffers hold what the
    descriptors say, and a solve of 200 iterations ends."""
    fake_device.run(fake, """
        ham, prm = S.hubbard_ring(8, 4.0), S.Params(tau=0.01, target_walkers=10**6, initial_walkers=1000)
        fake.fake_iteration(1000, 100, 300, 100, 5, 20)
        used = fake.fake_used()
        h = F.fciqmc_init(ham, prm)
        F.fciqmc_iterate(h, 200)
        assert F.fciqmc_estimators(h)["iteration"] == 200
        assert fake.fake_spawns() == 200 and fake.fake_faults() == 0 and fake.fake_graphs() > 0
        F.fciqmc_free(h)
        assert fake.fake_used() == used and fake.fake_graphs() == 0
    """)


@pytest.mark.parametrize("how", ["planned", "extensions", "option", "rebucket", "admission"])
def test_record_buffer_that_cannot_grow(fake, how):
    """A record buffer that could not be made larger is gone: the next call asks for it again
    (and fails again, or goes on when there is room) and launches nothing without it."""
    fake_device.run(fake, f"""
        how = {how!r}
        ham = S.hubbard_ring(8, 4.0)
        prm = S.Params(tau=0.01, target_walkers=10**6, initial_walkers=1000, det_capacity=1 << 20)
        fake.fake_iteration(1000, 100, 300, 100, 5, 20)
        h = F.fciqmc_batch_create(2, [ham], [prm])
        F.fciqmc_batch_iterate(h, 3)
        full, spawns = 64 << 30, fake.fake_spawns()
        tight = fake.fake_used() + (1 << 20)
        if how == "planned":          # the fullest bucket grows a hundredfold
            fake.fake_iteration(1000000, 1000, 30000, 1000, 5, 1000)
            F.fciqmc_batch_iterate(h, 1)
            spawns += 1
            fake.fake_capacity(tight)
            first = lambda: F.fciqmc_batch_iterate(h, 1)
        elif how == "extensions":     # records crowd into few buckets
            fake.fake_iteration(1000, 100, 300, 100, 5, 100000)
            F.fciqmc_batch_iterate(h, 1)
            spawns += 1
            fake.fake_extend(1 << 30)
            fake.fake_capacity(tight)
            first = lambda: F.fciqmc_batch_iterate(h, 1)
        elif how == "option":
            first = lambda: F.fciqmc_set_test_options(h, 1, -1, 1 << 40)
        elif how == "rebucket":       # room for the list, not for its buckets' record slots
            prm.target_walkers = 1 << 23
            fake.fake_capacity(fake.fake_used() + F.fciqmc_footprint_bytes(ham, prm))
            first = lambda: F.fciqmc_reserve(h, 1 << 24)
        else:
            prm.spawn_capacity = 1 << 40
            first = lambda: F.fciqmc_batch_admit(h, ham, prm)
        code = error(first)
        assert code == -2, code
        fake.fake_capacity(tight - (8 << 20))
        assert error(F.fciqmc_batch_iterate, h, 1) == -2
        assert fake.fake_spawns() == spawns and fake.fake_faults() == 0
        fake.fake_capacity(full)
        F.fciqmc_batch_iterate(h, 5)
        assert fake.fake_spawns() == spawns + 5 and fake.fake_faults() == 0
        F.fciqmc_free(h)
    """)


def test_chunk_maps_that_do_not_fit(fake):
    """A list re-bucketed into the last of the memory leaves none for the maps of its chunks:
    the next call asks for them again and launches nothing without them."""
    fake_device.run(fake, """
        ham = S.hubbard_ring(8, 4.0)
        prm = S.Params(tau=0.01, target_walkers=1 << 23, initial_walkers=1000, det_capacity=4096)
        fake.fake_iteration(1000, 100, 300, 100, 5, 20)
        h = F.fciqmc_init(ham, prm)
        F.fciqmc_iterate(h, 3)
        fake.fake_capacity(fake.fake_used() + F.fciqmc_footprint_bytes(ham, prm))
        assert error(F.fciqmc_reserve, h, 1 << 24) != 0
        for _ in range(2):
            assert error(F.fciqmc_iterate, h, 1) != 0
        assert fake.fake_spawns() == 3 and fake.fake_faults() == 0
        fake.fake_capacity(64 << 30)
        F.fciqmc_iterate(h, 5)
        assert fake.fake_spawns() == 8 and fake.fake_faults() == 0
        F.fciqmc_free(h)
        assert fake.fake_used() == 0
    """)


def test_refused_admission_leaves_its_slot(fake):
    """An admission refused for its record buffer leaves the slot free, the memory as it was
    and the other systems' slots at their own count."""
    fake_device.run(fake, """
        ham = S.hubbard_ring(8, 4.0)
        prm = S.Params(tau=0.01, target_walkers=10**6, initial_walkers=1000)
        fake.fake_iteration(1000, 100, 300, 100, 5, 20)
        h = F.fciqmc_batch_create(2, [ham], [prm])
        F.fciqmc_batch_iterate(h, 3)
        used = fake.fake_used()
        prm.spawn_capacity = 1 << 40
        assert error(F.fciqmc_batch_admit, h, ham, prm) == -2
        assert F.fciqmc_batch_active(h) == 1
        F.fciqmc_batch_iterate(h, 3)
        assert fake.fake_used() == used and fake.fake_faults() == 0
        prm.spawn_capacity = 0
        assert F.fciqmc_batch_admit(h, ham, prm) == 1
        F.fciqmc_batch_iterate(h, 3)
        assert fake.fake_faults() == 0
        F.fciqmc_free(h)
    """)


def test_captured_graphs_are_bounded(fake):
    """A solve whose population, births and call lengths keep changing meets hundreds of
    combinations of length and launch shape; the handle keeps the 64 used last."""
    fake_device.run(fake, """
        ham = S.hubbard_ring(8, 4.0)
        prm = S.Params(tau=0.01, target_walkers=10**9, initial_walkers=1000, det_capacity=1 << 23)
        h = F.fciqmc_init(ham, prm)
        most = 0
        for step in range(400):
            nw = 1000 << (step * 7 % 17)
            fake.fake_iteration(nw, 100, 300, 100, (step * 5 % 11) ** 6, 20)
            F.fciqmc_iterate(h, 2 + step * 13 % 40)
            most = max(most, fake.fake_graphs())
        assert most == 64, most
        assert fake.fake_faults() == 0
        F.fciqmc_free(h)
        assert fake.fake_graphs() == 0
    """)


def test_more_buckets_only_where_there_is_room(fake):
    """More buckets for a list of many records save time only: they are not made where their
    table fits into the device but would leave no room for their record slots."""
    fake_device.run(fake, """
        ham = S.hubbard_ring(8, 4.0)
        prm = S.Params(tau=0.01, target_walkers=10**6, initial_walkers=1000, det_capacity=1 << 20)
        fake.fake_iteration(1000000, 100000, 4000000, 100000, 5, 20)
        h = F.fciqmc_init(ham, prm)
        F.fciqmc_iterate(h, 1)
        split = 4000000 // 32 * 256 * 20 + 4000000 // 32 * 4
        fake.fake_capacity(fake.fake_used() + split + (12 << 20))
        F.fciqmc_iterate(h, 5)
        assert F.fciqmc_estimators(h)["table_slots"] == 1 << 20
        fake.fake_capacity(64 << 30)
        F.fciqmc_free(h)
        h = F.fciqmc_init(ham, prm)
        F.fciqmc_iterate(h, 1)
        F.fciqmc_iterate(h, 5)
        assert F.fciqmc_estimators(h)["table_slots"] >= 4000000 // 32 * 256
        assert fake.fake_faults() == 0
        F.fciqmc_free(h)
    """)

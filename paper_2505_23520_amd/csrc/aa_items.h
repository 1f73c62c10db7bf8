// Work items of a kernel whose work-groups take several, one after the other.  constexpr: the same code on the host.
#pragma once

namespace aa {

// The first item that exists of id, id + stride, id + 2 stride, .. below total: id becomes its number, x the item.  If there is
// none, id ends at total or beyond and x stays as it is: what a caller requests ahead for x is then still of an item that
// exists (an item that does not may name an address beyond the tensors: the first block of an empty last sequence).
template <class Item, class Of, class Exists>
constexpr bool next_item(unsigned& id, unsigned stride, unsigned total, Item& x, Of item_of, Exists exists) {
    for (; id < total; id += stride) {
        const Item y = item_of(id);
        if (exists(y)) {
            x = y;
            return true;
        }
    }
    return false;
}

}  // namespace aa

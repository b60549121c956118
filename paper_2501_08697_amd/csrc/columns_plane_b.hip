#include "columns_plane.hpp"

namespace apw {
template int columns_plane_n1<20>(const ColumnsCall &);
template int columns_plane_n1<24>(const ColumnsCall &);
template int columns_plane_n1<27>(const ColumnsCall &);
template int columns_plane_n1<30>(const ColumnsCall &);
}  // namespace apw
